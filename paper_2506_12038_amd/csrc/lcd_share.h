// How a decode launch shares its workgroups out over its layers, and the passes of the bucket kernel that this depends on.  Host code, no HIP.
#pragma once
#include <algorithm>
#include "lcd_internal.h"

namespace lcd {

// ---- passes of the bucket kernel (lcd_bucket.hip) -------------------------------------------------
constexpr int kBucketPass[] = {1, 2, 3, 7, 5, 10, 14};   // row tiles of a pass; all kernels have the first `lengths` of them
struct BucketRule {
    int waves;      // of a workgroup
    int operands;   // row tiles that a chunk's operands cost as much as
    int lengths;
    bool long_ties;
};

// Waves: 16 for one token of fp16 activations, 8 where more operands are held, with the same number for every pass (an output is the sum of the waves' sums:
// grouped, single and captured calls agree bit for bit).  One token of codes at 2 bits has registers for 16 too, but half of them would wait for nothing up to
// K = 2048; one row tile per workgroup, 8 / 16 waves, us: K = 1024 2.3 / 2.8, 2048 2.7 / 3.1, 4096 3.4 / 3.4, 8192 4.7 / 4.2, 28672 11.3 / 8.5; seven row tiles
// 4.1 / 5.0, 4.7 / 5.7, 6.7 / 6.9, 11.1 / 11.1.
constexpr int bucket_waves(int token_slots, bool int8_codes) { return token_slots == 1 && !int8_codes ? 16 : 8; }

// tokens: 1 (2 and 3 bits), 2 (2 bits), 3 and 4 (2 bits, INT8 codes)
constexpr BucketRule bucket_rule(int bits, int tokens, bool int8_codes)
{
    const int operands = tokens > 2 ? 4 : tokens == 2 && !int8_codes ? 2 : 1;
    return BucketRule{bucket_waves(tokens, int8_codes), operands, operands > 1 ? 7 : bits == 3 && !int8_codes ? 3 : 4, bits == 2 && operands == 1};
}

// Which of kBucketPass workgroups of up to `tiles` row tiles and kc chunks take.  Three row tiles at a time cover the latency of memory; longer passes
// make a step's operands less often (a wave's only chunk: once) -- but a slot without a row
// tile costs the addresses of its loads.  us, passes of 3 / 7: 2 bits, one token, 1792 row tiles, K = 8192 12.2 / 11.6, 3168, K = 4096 10.8 / 11.0;
// two tokens 13.9 / 11.9 (INT8 codes, K = 8192); four tokens, 3584, K = 8192, passes of 3 / 6 / 10 / 14: 36.5 / 29.6 / 27.8 / 25.3, 640, K = 5120 6.6 / 6.7 / 7.2 / 8.0.
// On a tie the longer pass (2 bits; one token, one and two of codes, three / seven, row tiles per workgroup: 5 x K = 5120 6.6 / 6.4 6.8 / 6.1 7.3 / 6.3, 11 x 8192 16.8 / 16.7
// 16.3 / 16.3 18.0 / 17.0, 22 x 5120 21.3 / 21.1 22.0 / 20.7 23.8 / 21.7; 70B MLP in one launch, 22 tiles 30.9 / 30.5), but not where three divides the row tiles (one
// token, 6 x 11008 13.2 / 13.8), nor 16 of them (x 8192 25.0 / 28.7: workgroups a power of two apart meet in the same memory channels).  Codes of 3 bits are as fast or faster
// with three up to K = 5120 (11 x 5120 18.3 / 18.9).
constexpr int bucket_pass(const BucketRule &rule, int tiles, int kc)
{
    if (kc <= rule.waves) return tiles < 3 ? tiles - 1 : 2;
    int best = 0;
    long long least = 0;
    for (int i = 0; i < rule.lengths; ++i) {
        const long long cost = (long long)((tiles + kBucketPass[i] - 1) / kBucketPass[i]) * (kBucketPass[i] + rule.operands);
        const bool tie = cost == least && rule.long_ties && tiles % 3 != 0 && tiles % 16 != 0 && kBucketPass[i] > 3;
        if (i == 0 || cost < least || tie) { best = i; least = cost; }
    }
    return best;
}

// ---- workgroups of the layers ---------------------------------------------------------------------
// A layer's time is that of its slowest workgroup: a fixed start-up, then one round of chunks (one for each wave) after the other.  In us.
constexpr int round_up_div(int a, int b) { return (a + b - 1) / b; }

struct DecodeCost {
    // the tokens and the narrow kernel: `held` row tiles a pass, 8 waves.  Fitted to single layers of
    // 4096 x t rows (t row tiles per workgroup), K = 4096 and 11008, 4 and 16 tokens; 2 bits, 16 tokens: K = 4096 t = 8, 10, 12
    // 15.0, 17.1, 19.0 us, 13 in two passes 25.4; K = 11008 t = 4, 5, 6 20.1, 23.0, 26.2.
    int held, blocks;
    double stage;             // of a round's activations
    // the bucket kernel (held = 0): a round's chunks each cost their operands once per pass
    BucketRule rule;
    double tile, chunk;

    int rounds(int kc) const { return round_up_div(kc, held ? 8 : rule.waves); }
    double round_tile(int bits) const { return held ? (bits == 2 ? 0.43 : bits == 3 ? 0.55 : 0.89) + 0.06 * blocks : tile; }
    // of a workgroup with t row tiles of a layer of kc chunks
    double time(int bits, int kc, int t) const
    {
        if (held) return round_up_div(t, held) * ((bits == 2 ? 3.7 : 5.0) + rounds(kc) * stage) + rounds(kc) * t * round_tile(bits);
        return 2.8 + rounds(kc) * (tile * t + chunk * round_up_div(t, kBucketPass[bucket_pass(rule, t, kc)]));
    }
};
inline DecodeCost tokens_cost(int held, int tokens, bool staged_ahead)
{
    const int blocks = round_up_div(tokens, 16);
    return DecodeCost{held, blocks, staged_ahead ? 0.1 * blocks : 0.08 + 0.035 * tokens, {}, 0.0, 0.0};
}
inline DecodeCost bucket_cost(int bits, int tokens, bool int8_codes)
{
    return DecodeCost{0, 0, 0.0, bucket_rule(bits, tokens, int8_codes), bits == 3 ? (int8_codes ? 0.45 : 1.05) : tokens > 1 ? 0.35 : int8_codes ? 0.3 : 0.6,
                      tokens == 1 ? 0.1 : int8_codes && tokens > 2 ? 0.15 * tokens : 0.2};
}

struct LayerShape { int tiles, kc, bits; };   // row tiles, chunks, index width
inline bool operator==(const LayerShape &a, const LayerShape &b) { return a.tiles == b.tiles && a.kc == b.kc && a.bits == b.bits; }

// Shares `grid` workgroups (at least `count`) out over the layers so that the slowest one is as fast as it can be.  A workgroup's time grows with its
// row tiles, but for steps of the bucket kernel's passes, whose length depends on them (21 row tiles may take longer than 22).
inline void share_workgroups(const DecodeCost &cost, const LayerShape *layers, int count, int grid, int *out)
{
    auto time = [&](int i, int t) { return cost.time(layers[i].bits, layers[i].kc, t); };
    int like[kMaxGroup];      // the first layer of the same shape: its answer is this one's
    for (int i = 0; i < count; ++i)
        for (like[i] = 0; !(layers[like[i]] == layers[i]);) ++like[i];
    // smallest number of workgroups with which layer i takes at most T (0: not even one per tile does): the largest share of row tiles first
    auto need = [&](int i, double T) {
        const int tiles = layers[i].tiles;
        const double most = T / (cost.rounds(layers[i].kc) * cost.round_tile(layers[i].bits));   // more row tiles take longer than T by themselves
        for (int t = most < tiles ? (int)most : tiles; t > 0;) {
            const int n = round_up_div(tiles, t), share = round_up_div(tiles, n);
            if (time(i, share) <= T) return n;
            t = share - 1;
        }
        return 0;
    };
    auto fits = [&](double T, int *n) {
        int sum = 0;
        for (int i = 0; i < count; ++i) {
            n[i] = like[i] < i ? n[like[i]] : need(i, T);
            if (n[i] == 0) return false;
            sum += n[i];
        }
        return sum <= grid;
    };
    // the smallest common finish time the grid can reach
    double t_lo = 0.0, t_hi = 0.0;
    bool alike = true;
    for (int i = 0; i < count; ++i) alike = alike && like[i] == 0;
    if (alike) {              // equal parts (q, k, v; gate, up: 2.5 and 1.6 us of host time by bisection, 0.2 so)
        const int tiles = layers[0].tiles, share = round_up_div(tiles, std::min(tiles, grid / count));
        t_hi = time(0, share);
        for (int t = share + 1; !cost.held && t <= tiles && t * cost.rounds(layers[0].kc) * cost.tile < t_hi; ++t)
            if (round_up_div(tiles, round_up_div(tiles, t)) == t) t_hi = std::min(t_hi, time(0, t));   // (some number of workgroups has this share)
    } else {                  // bisection between "one workgroup per tile everywhere" and "one workgroup per layer"
        for (int i = 0; i < count; ++i) {
            if (like[i] < i) continue;
            t_lo = std::max(t_lo, time(i, 1));
            t_hi = std::max(t_hi, time(i, layers[i].tiles));
        }
        int trial[kMaxGroup];
        if (fits(t_lo, trial)) t_hi = t_lo;
        for (int it = 0; it < 24 && t_hi - t_lo > 0.02; ++it) {
            const double mid = 0.5 * (t_lo + t_hi);
            if (fits(mid, trial)) t_hi = mid; else t_lo = mid;
        }
    }
    fits(t_hi, out);
    // spare workgroups: to the layer that is slowest then, as many as make its largest share smaller
    int used = 0;
    double now[kMaxGroup];
    bool more_helps[kMaxGroup];
    for (int i = 0; i < count; ++i) {
        used += out[i];
        now[i] = like[i] < i ? now[like[i]] : time(i, round_up_div(layers[i].tiles, out[i]));
        more_helps[i] = out[i] < layers[i].tiles;
    }
    while (used < grid) {
        int i = -1;
        for (int q = 0; q < count; ++q)
            if (more_helps[q] && (i < 0 || now[q] > now[i])) i = q;
        if (i < 0) break;
        const int tiles = layers[i].tiles, share = round_up_div(tiles, out[i]);      // (at least two: fewer workgroups than tiles)
        const int more = std::min(grid - used, round_up_div(tiles, share - 1) - out[i]);
        const double then = time(i, round_up_div(tiles, out[i] + more));
        more_helps[i] = then <= now[i] && out[i] + more < tiles;
        if (then > now[i]) continue;
        out[i] += more;
        used += more;
        now[i] = then;
    }
}

}  // namespace lcd
