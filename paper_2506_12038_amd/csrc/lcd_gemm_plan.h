// Which tiles a launch of the wide prefill kernel takes, which workgroup takes which tile, and which of the kernel's two forms takes a layer.
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

// ---- tiles -------------------------------------------------------------------------------------------
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

struct WideLayer { int N, K; };
// Rounds of workgroups over the compute units, the columns of more blocks first.  Each round takes the time of its longest workgroup alone, or what a full chip
// would take of it, smoothed.  more_us: shorter workgroups of another kind that follow in the same launch, in us of the whole chip: they fill the last round.
inline double wide_time(const WideTiles &t, const WideLayer *layers, int count, int bits, int cus, double more_us = 0.0)
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
inline WideTiles choose_wide(bool whole, const WideLayer *layers, int count, int token_blocks, int bits, int cus, double *time = nullptr, double more_us = 0.0)
{
    WideTiles best{};
    double least = 0.0;
    for (int form = whole ? kWhole256 : kHalves128; form <= (whole ? kWhole256 : kHalves256); ++form) {
        const int most = whole ? 8 : 4, fewest = whole ? 5 : 2;
        for (int b = most; b >= fewest; --b) {
            const WideTiles t = wide_columns(form, token_blocks, (token_blocks + b - 1) / b);
            if (whole && t.blocks < 5) continue;
            const double us = wide_time(t, layers, count, bits, cus, more_us);
            if (best.columns == 0 || us < least) { best = t; least = us; }
        }
    }
    if (time) *time = least;
    return best;
}

// Which form takes a layer.  They add in different orders, so this looks at the layer and the tokens alone.
inline bool whole_takes(int M, int N, int K, int bits)
{
    const WideLayer pair[2] = {{N, K}, {N, K}};
    const int blocks = (M + 31) / 32;
    if (blocks < 5) return false;
    double whole[2], halves[2];
    for (int n = 0; n < 2; ++n) {
        if (choose_wide(true, pair, n + 1, blocks, bits, 256, &whole[n]).columns == 0) return false;
        choose_wide(false, pair, n + 1, blocks, bits, 256, &halves[n]);
    }
    return whole[0] * whole[1] < halves[0] * halves[1] && whole[0] < 1.1 * halves[0];
}

}  // namespace lcd
