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
};

// Waves: 16 for one token of fp16 activations, 8 where more operands are held, with the same number for every pass (an output is the sum of the waves' sums:
// grouped, single and captured calls agree bit for bit).  One token of codes at 2 bits has registers for 16 too, but they win on one or two row tiles
// of long rows alone, 8 / 16 waves, us: one row tile per workgroup, K = 1024 2.3 / 2.8, 2048 2.7 / 3.1, 4096 3.4 / 3.4, 8192 4.7 / 4.2, 28672 11.3 / 8.5; best pass of 4 row
// tiles, K = 4096 4.7 / 5.1, 8192 7.1 / 7.5, of 10 8.6 / 8.7, 14.9 / 15.5.
constexpr int bucket_waves(int token_slots, bool int8_codes) { return token_slots == 1 && !int8_codes ? 16 : 8; }

// tokens: 1 (2 and 3 bits), 2 (2 bits), 3 and 4 (2 bits, INT8 codes)
constexpr BucketRule bucket_rule(int bits, int tokens, bool int8_codes)
{
    const int lengths = tokens > 2 || (tokens == 2 && !int8_codes) ? 7 : bits == 3 && !int8_codes ? 3 : 5;   // (longer ones spill or lose)
    return BucketRule{bucket_waves(tokens, int8_codes), tokens > 2 ? 4 : bits == 2 ? 2 : 1, lengths};
}

// Which of kBucketPass workgroups of up to `tiles` row tiles and kc chunks take.  Three row tiles at a time cover the latency of memory; longer passes
// make a step's operands less often (a wave's only chunk: once), but a place without a row
// tile costs the addresses of its loads.  One launch, weights from memory, us:
//   passes of 2 / 3 / 5 / 7   one token of codes, 2 bits: 4 row tiles per workgroup, K = 4096 5.3 5.4 4.7 4.9; 8 tiles 8.3 7.7 7.3 8.2; 10, 2304 8.1 7.4 6.3 6.5; 16, 5120 18.4 16.7 16.0 15.7;
//     12, 8192 19.7 17.2 18.1 17.7    two tokens: 4, 4096 5.9 5.9 5.2 5.2; 10, 8192 19.0 17.2 15.4 15.9    fp16: 10, 5120 11.4 10.9 10.2 10.9; 8, 4352 9.0 8.3 8.3 8.8    codes, 3 bits: 10,
//     5120 17.9 17.2 15.9 17.5; 8, 8192 23.3 21.5 21.2 23.3
//   four tokens of codes, 14 row tiles, K = 8192, passes of 3 / 6 / 10 / 14: 36.5 / 29.6 / 27.8 / 25.3, 2.5 row tiles, K = 5120 6.6 / 6.7 / 7.2 / 8.0
// The rule's choice took 1.010 times the best pass's time in the mean over 3 to 28 row tiles and K = 2304 to 11008 with one token of codes at 2 bits, 1.004 with two, 1.003 with
// fp16 activations, 1.010 at 3 bits.
constexpr int bucket_pass(const BucketRule &rule, int tiles, int kc)
{
    if (kc <= rule.waves) return tiles < 3 ? tiles - 1 : 2;
    int best = -1;
    long long least = 0;
    for (int i = 0; i < rule.lengths; ++i) {
        if (rule.lengths > 3 && kBucketPass[i] < 3 && tiles > kBucketPass[i]) continue;   // several passes of one or two lose wherever three or more are to be had
        const long long cost = (long long)((tiles + kBucketPass[i] - 1) / kBucketPass[i]) * (kBucketPass[i] + rule.operands);
        if (best < 0 || cost < least) { best = i; least = cost; }
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
    // the bucket kernel (held = 0): a round's chunks each cost their operands once per pass (a wave's only chunk: once), passes of `pass` row tiles,
    // every place of which counts, or (0) of the length that suits the row tiles of a workgroup
    BucketRule rule;
    double tile, chunk;
    int pass;
    double empty;             // what a place without a row tile costs of a row tile's time where it is in a workgroup's only pass (in the last of several: all)
    static constexpr double kStart = 2.8;

    int rounds(int kc) const { return round_up_div(kc, held ? 8 : rule.waves); }
    double round_tile(int bits) const { return held ? (bits == 2 ? 0.43 : bits == 3 ? 0.55 : 0.89) + 0.06 * blocks : tile; }
    // of a workgroup with t row tiles of a layer of kc chunks
    double time(int bits, int kc, int t) const
    {
        if (held) return round_up_div(t, held) * ((bits == 2 ? 3.7 : 5.0) + rounds(kc) * stage) + rounds(kc) * t * round_tile(bits);
        if (pass) {
            const int passes = round_up_div(t, pass);
            return kStart + rounds(kc) * tile * (rule.operands * (kc > rule.waves ? passes : 1) + (t < pass ? t + empty * (pass - t) : pass * passes));
        }
        return even_time(bits, kc, t);
    }
    // the same where places without a row tile are free
    double even_time(int bits, int kc, int t) const
    {
        if (held) return time(bits, kc, t);
        return kStart + rounds(kc) * (tile * t + chunk * round_up_div(t, pass ? pass : kBucketPass[bucket_pass(rule, t, kc)]));
    }
};
inline DecodeCost tokens_cost(int held, int tokens, bool staged_ahead)
{
    const int blocks = round_up_div(tokens, 16);
    return DecodeCost{held, blocks, staged_ahead ? 0.1 * blocks : 0.08 + 0.035 * tokens, {}, 0.0, 0.0, 0, 0.0};
}
inline DecodeCost bucket_cost(int bits, int tokens, bool int8_codes)
{
    return DecodeCost{0, 0, 0.0, bucket_rule(bits, tokens, int8_codes), bits == 3 ? (int8_codes ? 0.45 : 1.05) : tokens > 1 ? 0.35 : int8_codes ? 0.3 : 0.6,
                      tokens == 1 ? 0.1 : int8_codes && tokens > 2 ? 0.15 * tokens : 0.2, 0, int8_codes ? 0.3 : 1.0};
}

struct LayerShape { int tiles, kc, bits; };   // row tiles, chunks, index width
inline bool operator==(const LayerShape &a, const LayerShape &b) { return a.tiles == b.tiles && a.kc == b.kc && a.bits == b.bits; }

// Shares `grid` workgroups (at least `count`) out over the layers so that the slowest one is as fast as it can be; returns its time.  A workgroup's time
// grows with its row tiles, but for steps where the length of the bucket kernel's passes depends on them (21 row tiles may take longer than 22).
inline double share_workgroups(const DecodeCost &cost, const LayerShape *layers, int count, int grid, int *out)
{
    auto time = [&](int i, int t) { return cost.time(layers[i].bits, layers[i].kc, t); };
    int like[kMaxGroup];      // the first layer of the same shape: its answer is this one's
    for (int i = 0; i < count; ++i)
        for (like[i] = 0; !(layers[like[i]] == layers[i]);) ++like[i];
    // smallest number of workgroups with which layer i takes at most T (0: not even one per tile does): the largest share of row tiles first
    auto need = [&](int i, double T) {
        const int tiles = layers[i].tiles;
        if (cost.pass) {
            const double unit = cost.rounds(layers[i].kc) * cost.tile, work = (T - DecodeCost::kStart) / unit + 1e-9;
            const bool once = layers[i].kc <= cost.rule.waves;     // (a wave makes the operands of its only chunk once)
            const int passes = (int)std::min<double>(once ? (work - cost.rule.operands) / cost.pass : work / (cost.pass + cost.rule.operands), tiles);
            int share = passes * cost.pass;
            if (passes <= 0 && cost.empty < 1.0) share = (int)std::max(0.0, (work - cost.rule.operands - cost.empty * cost.pass) / (1.0 - cost.empty));
            return share > 0 ? round_up_div(tiles, share) : 0;
        }
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
    auto even_time = [&](int i, int n) { return cost.even_time(layers[i].bits, layers[i].kc, round_up_div(layers[i].tiles, n)); };
    int used = 0;
    double now[kMaxGroup];
    bool more_helps[kMaxGroup];
    for (int i = 0; i < count; ++i) {
        used += out[i];
        now[i] = like[i] < i ? now[like[i]] : even_time(i, out[i]);
        more_helps[i] = out[i] < layers[i].tiles;
    }
    while (used < grid) {
        int i = -1;
        for (int q = 0; q < count; ++q)
            if (more_helps[q] && (i < 0 || now[q] > now[i])) i = q;
        if (i < 0) break;
        const int tiles = layers[i].tiles, share = round_up_div(tiles, out[i]);      // (at least two: fewer workgroups than tiles)
        const int more = std::min(grid - used, round_up_div(tiles, share - 1) - out[i]);
        const double then = even_time(i, out[i] + more);
        more_helps[i] = then <= now[i] && out[i] + more < tiles;
        if (then > now[i]) continue;
        out[i] += more;
        used += more;
        now[i] = then;
    }
    return t_hi;
}

// The bucket kernel's shares; returns the place in kBucketPass of the launch's passes.  Layers of different shapes get shares that go with the passes, of the
// length that makes the slowest layer fastest.  70B MLP in one launch, one and two tokens of codes, passes of five, shares
// without a look at the passes 34.5 35.0 us, so 30.4 31.5.  Seven layers of a block, with places in an only pass / and operands of an only chunk
// in each pass counted whole, so: 7B, one token of codes, 2 and 3 bits 10.7 18.4, 10.3 18.1; 3072 / 8192, fp16 and codes of 3 bits 7.2 11.5, 6.8 9.6.
inline int share_bucket(int bits, int tokens, bool int8_codes, const LayerShape *layers, int count, int grid, int *out)
{
    DecodeCost cost = bucket_cost(bits, tokens, int8_codes);
    const BucketRule &rule = cost.rule;
    bool alike = true;
    int widest = 0, most = 1;
    for (int i = 0; i < count; ++i) {
        alike = alike && layers[i] == layers[0];
        widest = std::max(widest, layers[i].kc);
    }
    if (!alike && rule.lengths == 5 && widest > rule.waves) {
        int best = -1, trial[kMaxGroup];
        double least = 0.0;
        for (int i : {2, 4, 3}) {     // three, five, seven
            cost.pass = kBucketPass[i];
            const double time = share_workgroups(cost, layers, count, grid, trial);
            if (best >= 0 && time >= least) continue;
            best = i;
            least = time;
            std::copy(trial, trial + count, out);
        }
        for (int i = 0; i < count; ++i) most = std::max(most, round_up_div(layers[i].tiles, out[i]));
        return most < 3 ? most - 1 : best;
    }
    if (count == 1) out[0] = grid;
    else share_workgroups(cost, layers, count, grid, out);
    for (int i = 0; i < count; ++i) most = std::max(most, round_up_div(layers[i].tiles, out[i]));
    return bucket_pass(rule, most, widest);
}

}  // namespace lcd
