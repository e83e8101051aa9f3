// Which prefill kernel takes a layer, which tiles a launch of the wide and of the split kernel takes, and which workgroup takes which wide tile.
// Host code that any C++ compiler takes, but for wide_tile_of, which the kernel runs too.
#pragma once
#include <cmath>
#include "lcd_internal.h"

#ifdef __HIPCC__
#define LCD_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define LCD_HOST_DEVICE inline
#endif

namespace lcd {

struct LayerSize { int N, K; };

// ---- kernels -----------------------------------------------------------------------------------------
// Which kernel takes a layer.  The rules look at the layer and the number of tokens alone, never at the group it is
// called in: the kernels add in different orders, and a layer's result must not depend on its neighbours.
// Up to 16 tokens the decode kernels (the dequantising one, except for INT8 codes with 2-bit indices).  Up to 32 tokens the tokens kernel, which needs no smoothing launch,
// also keeps the small layers.  One call with 32 tokens, weights from memory, tokens kernel / split kernel, 2, 3 and 4 bits: 2048 x 2048
// 6.4/8.1 6.7/8.9 7.0/9.3 us, 2048 x 4096 8.3/10.6 8.7/11.4 9.3/11.9, 11008 x 1024 7.1/8.7 7.9/9.0 7.7/9.8, 28672 x 512 11.9/12.0 13.2/12.4 16.6/13.3;
// beyond the line 4096 x 4096 8.9/10.9 9.4/11.6 10.2/12.5, 6144 x 4096 11.6/11.0 12.5/11.8 15.1/13.0, 8192 x 4096 11.7/11.2 13.0/12.1 15.9/13.8.  A
// layer of 4096 x 4096 alone would gain from the tokens kernel too; three of them in one call, which must take the same kernel, are
// 12288 x 4096 to it and would lose.
inline bool decode_takes(int M, int N, int K)
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
inline bool narrow_takes(int M, int N, int K, int bits)
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
inline bool split_takes(int M, int N, int K, int bits)
{
    const long long blocks = (M + 127) / 128, rows64 = (N + 63) / 64;
    return rows64 * blocks <= (bits == 2 ? 224 : 256) && blocks * 128 * K * 2 < (1ll << 32);
}


// ---- wide tiles --------------------------------------------------------------------------------------
// A tile of the wide kernel (lcd_gemm_wide.h) is 256 rows (or 128) x up to 8 blocks of 32 tokens.  The blocks of a call are dealt out to columns of tiles as
// evenly as they go: `big` columns of `blocks`, then columns of one block less.
struct WideTiles {
    int form;        // rows: see below
    int blocks, big, columns;
};
// halves: 8 waves, K in two halves, up to 4 blocks; whole: 4 waves, all of K each, 5 to 8 blocks (4 where 5 are not reached everywhere)
enum { kHalves128, kHalves256, kWhole256 };
inline int wide_rows(int form) { return form == kHalves128 ? 128 : 256; }

inline WideTiles wide_columns(int form, int token_blocks, int columns)
{
    const int blocks = (token_blocks + columns - 1) / columns;
    return WideTiles{form, blocks, token_blocks - columns * (blocks - 1), columns};
}

// ---- numbering ------------------------------------------------------------------------------------------
// XCD-aware tile order.  Workgroup ids go round-robin over the 8 XCDs, each with its own L2.  The tiles of a layer's columns of one width are numbered
// token-block-major and cut into 8 contiguous runs, one per XCD, so that the workgroups that are resident on an XCD at the same time share one or two columns'
// activations.  The wider columns come first (of every layer).  Runs differ by one tile; which XCDs have the longer ones goes round from one set of columns
// to the next, so that no XCD has more than one tile more than another (with all runs of a set as long as its longest, 250 tiles -- two layers of 6400 x 3072,
// 1244 tokens -- took a second round on six XCDs: 133 us instead of 89).
struct WideTileAt { int layer, second, tile; };    // layer < 0: a workgroup without a tile; second: in the columns of one block less
// batch.p[i].tiles[second]: a layer's tiles in either set of columns
template <class Batch>
LCD_HOST_DEVICE WideTileAt wide_tile_of(const Batch &batch, uint32_t block)
{
    const uint32_t xcd = block % kXcds;
    uint32_t pos = block / kXcds, turn = 0;
    for (int second = 0; second < 2; ++second)
        for (int i = 0; i < batch.count; ++i) {
            const uint32_t tiles = batch.p[i].tiles[second], rest = tiles % kXcds;
            const uint32_t ones = (1u << rest) - 1, longer = (ones << turn | ones >> (kXcds - turn)) & 255u;     // XCDs with a run of one more
            const uint32_t run = tiles / kXcds + (longer >> xcd & 1);
            if (pos < run) return WideTileAt{i, second, (int)(xcd * (tiles / kXcds) + __builtin_popcount(longer & ((1u << xcd) - 1)) + pos)};
            pos -= run;
            turn = (turn + rest) % kXcds;
        }
    return WideTileAt{-1, 0, 0};
}

// ---- time ---------------------------------------------------------------------------------------------
// A workgroup's time: a start, and a part per column of K that depends on how much of the chip multiplies: alone it is the matrix pipe's (or the
// dequantiser's) at 2.3 GHz, on a full chip the power management's.  Fitted to single rounds of K = 4096 and 11008 and to full rounds of K = 8192.
struct WideTime { double start_us, column_ns[3], full_ns[3]; };     // 2, 3, 4 bits
constexpr WideTime kWideTime[3][8] = {
    {{0.5, {3.9, 4.3, 5.5}, {3.4, 4.0, 5.4}}, {0.5, {3.8, 4.4, 5.5}, {4.2, 5.0, 6.0}}, {2.0, {3.8, 4.4, 5.2}, {5.2, 5.8, 6.7}}, {3.2, {4.05, 4.7, 5.4}, {6.6, 7.0, 8.0}}},
    {{0.5, {5.0, 5.6, 7.9}, {5.3, 6.2, 8.6}}, {0.5, {5.35, 6.4, 8.7}, {6.8, 8.0, 11.2}}, {2.7, {6.0, 6.9, 9.2}, {9.3, 10.2, 12.3}}, {4.3, {7.5, 7.85, 10.0}, {11.7, 12.4, 15.6}}},
    {{}, {}, {}, {3.5, {8.3, 9.4, 12.0}, {12.2, 13.0, 15.4}}, {4.0, {10.05, 10.7, 12.9}, {15.0, 15.6, 17.5}}, {4.7, {11.8, 12.4, 14.3}, {17.5, 18.1, 19.9}},
     {5.5, {13.3, 13.85, 15.5}, {20.1, 20.8, 22.5}}, {6.9, {14.8, 15.2, 16.6}, {22.6, 23.1, 24.8}}},
};

// Rounds of workgroups over the compute units, the columns of more blocks first.  Each round takes the time of its longest workgroup alone, or what a full chip
// would take of it, smoothed.  more_us: shorter workgroups of another kind that follow in the same launch, in us of the whole chip: they fill the last round.
inline double wide_time(const WideTiles &t, const LayerSize *layers, int count, int bits, int cus, double more_us = 0.0)
{
    double us = 2.5, longest = 0.0, energy = 0.0, all = 0.0;
    int room = cus;
    auto round = [&] { const double a = longest * longest, b = energy / cus * (energy / cus); us += std::sqrt(std::sqrt(a * a + b * b)); longest = energy = 0.0; room = cus; };
    for (int part = 0; part < 2; ++part) {
        const int columns = part ? t.columns - t.big : t.big, blocks = t.blocks - part;
        if (columns <= 0 || blocks <= 0) continue;
        const WideTime &w = kWideTime[t.form][blocks - 1];
        for (int i = 0; i < count; ++i) {
            const double alone = w.start_us + 1e-3 * w.column_ns[bits - 2] * layers[i].K, full = w.start_us + 1e-3 * w.full_ns[bits - 2] * layers[i].K;
            long long tiles = (long long)((layers[i].N + wide_rows(t.form) - 1) / wide_rows(t.form)) * columns;
            all += tiles * full;
            while (tiles > 0) {
                if (room == cus && tiles >= 2 * cus) {       // rounds alike
                    const long long rounds = tiles / cus - 1;
                    const double a = alone * alone, b = full * full;
                    us += rounds * std::sqrt(std::sqrt(a * a + b * b));
                    tiles -= rounds * cus;
                }
                const int take = tiles < room ? (int)tiles : room;
                longest = alone > longest ? alone : longest;
                energy += take * full;
                tiles -= take;
                room -= take;
                if (room == 0) round();
            }
        }
    }
    if (room < cus) round();
    const double together = 2.5 + all / cus + more_us;
    return more_us > 0.0 && together > us ? together : us;
}

// The tiles with the least time of those that a form of the kernel has.
inline WideTiles choose_wide(bool whole, const LayerSize *layers, int count, int token_blocks, int bits, int cus, double *time = nullptr)
{
    WideTiles best{};
    double least = 0.0;
    for (int form = whole ? kWhole256 : kHalves128; form <= (whole ? kWhole256 : kHalves256); ++form) {
        const int most = whole ? 8 : 4, fewest = whole ? 5 : 2;
        for (int b = most; b >= fewest; --b) {
            const WideTiles t = wide_columns(form, token_blocks, (token_blocks + b - 1) / b);
            if (whole && t.blocks < 5) continue;
            const double us = wide_time(t, layers, count, bits, cus);
            if (best.columns == 0 || us < least) { best = t; least = us; }
        }
    }
    if (time) *time = least;
    return best;
}

// Which form takes a layer.  They add in different orders, so this looks at the layer and the tokens alone: whole where the model has one such layer
// and two of them in a launch faster in the product of both, and one layer no more than a tenth slower.  Time over the better form's for a layer on its own
// / three alike in a call, smoothing included, mean of 324 sizes (129 to 2048 tokens, 1024 to 28672 rows, K = 1024 to 11008, 2, 3 and 4 bits): this rule 1.002 / 1.035 (at
// most 1.10 / 1.29), without the tenth 1.001 / 1.040, halves always 1.022 / 1.060, whole wherever there are five blocks 1.30 / 1.033.  Whole / halves, us:
//   4096 x 4096    2048 tokens, 3 bits  68.6/66.8, three 173/180      1500 tokens, 4 bits  66.8/62.1, three 153/169
//   11008 x 4096    333 tokens, 2 bits  58.7/36.3, three 116/93       2048 tokens, 3 bits 160/168, three 456/497
//   4096 x 11008   1500 tokens, 4 bits 164/150, three 390/427         2048 tokens, 3 bits 172/165, three 446/454
//   8192 x 8192     333 tokens, 4 bits 129/60, three 151/172          2048 tokens, 4 bits 232/267, three 659/765
inline bool whole_takes(int M, int N, int K, int bits)
{
    const LayerSize pair[2] = {{N, K}, {N, K}};
    const int blocks = (M + 31) / 32;
    if (blocks < 5) return false;
    double whole[2], halves[2];
    for (int n = 0; n < 2; ++n) {
        if (choose_wide(true, pair, n + 1, blocks, bits, 256, &whole[n]).columns == 0) return false;
        choose_wide(false, pair, n + 1, blocks, bits, 256, &halves[n]);
    }
    return whole[0] * whole[1] < halves[0] * halves[1] && whole[0] < 1.1 * halves[0];
}

// The kernel of a layer.  whole: whole_takes, or a copy of its answers.
enum PrefillKernel { kDecodeKernels, kNarrowKernel, kSplitKernel, kWideHalves, kWideWhole };
inline PrefillKernel prefill_kernel(int M, int N, int K, int bits, bool (*whole)(int, int, int, int) = whole_takes)
{
    if (decode_takes(M, N, K)) return kDecodeKernels;
    if (narrow_takes(M, N, K, bits)) return kNarrowKernel;
    if (split_takes(M, N, K, bits)) return kSplitKernel;
    return whole(M, N, K, bits) ? kWideWhole : kWideHalves;
}

// ---- split tiles --------------------------------------------------------------------------------------
// Tile of a launch of the split kernel: rounds of workgroups over the compute units times the time of one workgroup.  Measured
// in single rounds (K = 4096 and 11008): a fixed part, and a part per column that is bound by the activations' way into LDS
// (75..98 GB/s per compute unit; 32 tokens x 64 rows: by the dequantiser).  In launches of several rounds every tile takes longer
// than that (the rounds share the L2), but their order holds: 177 launches timed with each of the six tiles (1 to 3 layers of 1024..13824
// rows, K = 2048..11008, 33..512 tokens, 2, 3 and 4 bits) took 1.002 times the best tile's time in the mean, 1.03 at the ninth decile,
// 1.14 at most (three layers of 2048 x 2048, 512 tokens, 3 bits: 32.8 against 28.9 us).
struct SplitTile { int pairs, blocks; double fixed_us, column_ns[3]; };   // column_ns: 2, 3, 4 bits
constexpr SplitTile kSplitTiles[] = {
    {2, 4, 3.0, {2.58, 2.70, 3.13}}, {2, 3, 2.5, {2.13, 2.40, 3.05}}, {2, 2, 2.0, {1.56, 1.74, 2.33}},
    {2, 1, 1.5, {1.34, 1.66, 2.58}}, {1, 2, 1.5, {1.48, 1.60, 1.69}}, {1, 1, 1.3, {0.79, 0.88, 1.17}},
};
// time of all workgroups of a tile's launch one after the other, and their number
inline double split_work(const LayerSize *layers, int count, const SplitTile &t, int M, int bits, double &wgs)
{
    double work = 0.0;
    wgs = 0.0;
    for (int q = 0; q < count; ++q) {
        const double n = (double)((layers[q].N + 32 * t.pairs - 1) / (32 * t.pairs)) * ((M + 32 * t.blocks - 1) / (32 * t.blocks));
        wgs += n;
        work += n * (t.fixed_us + 1e-3 * t.column_ns[bits - 2] * layers[q].K);
    }
    return work;
}
inline const SplitTile &choose_split_tile(const LayerSize *layers, int count, int M, int bits, int cus)
{
    const SplitTile *best = nullptr;
    double best_time = 0.0;
    for (const SplitTile &t : kSplitTiles) {
        double wgs;
        const double work = split_work(layers, count, t, M, bits, wgs), time = __builtin_ceil(wgs / cus) * work / wgs;
        if (!best || time < best_time) { best = &t; best_time = time; }
    }
    return *best;
}
// Next to wide tiles there are no rounds of their own to fill: the tile with the least work of the two that cost least per output.
inline const SplitTile &choose_mixed_tile(const LayerSize *layers, int count, int M, int bits)
{
    double wgs;
    return split_work(layers, count, kSplitTiles[0], M, bits, wgs) <= split_work(layers, count, kSplitTiles[1], M, bits, wgs) ? kSplitTiles[0] : kSplitTiles[1];
}


// ---- the matrix launches of a call ---------------------------------------------------------------------
// The launches of a call's split layers and wide layers in halves: one for both kinds (lcd_gemm_mixed.hip: wide tiles of 4 blocks, or of 3 throughout), whose
// split tiles fill the wide tiles' last round, wherever the tokens give such tiles; else one each with the tiles that suit it best.  357 groups with both
// kinds and such tiles (blocks of 7 layers, q, k, v with fewer rows in k and v, random groups of 2 to 8 layers; 97 to 1100 tokens; 2, 3 and 4 bits): one launch
// takes 1.003 times the better way's time in the mean, 1.10 at most (4944 + 1200 rows, K = 4096, 531 tokens, 4 bits: 53.5 us, apart 48.8), apart
// 1.088 and 1.39 (q, k, v of 5120 + 1280 + 1280 rows, K = 5120, 500 tokens, 3 bits 51 and 56; all of a 7B block, 333 tokens, 3 bits 166 and 194).  A model's
// choice between the two was worse: 1.02.
struct MatrixLaunches {
    WideTiles halves;
    const SplitTile *split;
    bool together;
};
inline bool mixed_has(const WideTiles &t) { return t.blocks == 4 || (t.blocks == 3 && t.big == t.columns); }
inline MatrixLaunches plan_launches(const LayerSize *halves, int halves_count, const LayerSize *split, int split_count, int M, int bits, int cus)
{
    const int token_blocks = (M + 31) / 32;
    MatrixLaunches l{};
    if (halves_count > 0 && split_count > 0) {
        const SplitTile &next = choose_mixed_tile(split, split_count, M, bits);
        double wgs, least = 0.0;
        const double more_us = 1.5 * split_work(split, split_count, next, M, bits, wgs) / cus;      // (next to wide tiles: 1.5 times what they take in a round of their own)
        for (int form = kHalves128; form <= kHalves256; ++form)
            for (int b = 4; b >= 3; --b) {
                const WideTiles t = wide_columns(form, token_blocks, (token_blocks + b - 1) / b);
                if (!mixed_has(t)) continue;
                const double us = wide_time(t, halves, halves_count, bits, cus, more_us);
                if (!l.together || us < least) { l = MatrixLaunches{t, &next, true}; least = us; }
            }
        if (l.together) return l;
    }
    if (halves_count > 0) l.halves = choose_wide(false, halves, halves_count, token_blocks, bits, cus);
    if (split_count > 0) l.split = &choose_split_tile(split, split_count, M, bits, cus);
    return l;
}

}  // namespace lcd
