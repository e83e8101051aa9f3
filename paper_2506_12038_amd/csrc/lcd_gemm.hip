// Prefill path (M >= 17; any M >= 1 accepted) of the smoothed table-lookup product, gfx950: the wide kernel
// (lcd_gemm_wide.h) and the launcher of all prefill kernels.
#include <hip/hip_runtime.h>
#include <algorithm>
#include "lcd_gemm_common.h"
#include "lcd_launch.h"

namespace lcd {

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
    LayerSize sizes[3][kMaxGroup];
    GroupItem small[kMaxGroup], narrow[kMaxGroup];
    int small_count = 0, narrow_count = 0;       // the decode kernels' layers, the narrow kernel's
    size_t offset = 0;
    for (int q = 0; q < count; ++q) {
        const GroupItem &it = items[order[q]];
        const PrefillKernel kernel = prefill_kernel(M, it.N, it.K, bits, wide_whole);
        if (kernel == kDecodeKernels) { small[small_count++] = it; continue; }
        if (kernel == kNarrowKernel) { narrow[narrow_count++] = it; continue; }
        uint8_t *xs = nullptr;
        for (int d = 0; d < distinct && !xs; ++d)
            if (sm[d].x == it.x && sm[d].s == it.s && sm[d].K == it.K && sm[d].s_q == it.act_scale) xs = static_cast<uint8_t *>(sm[d].xs);
        if (!xs) {
            xs = static_cast<uint8_t *>(workspace) + offset;
            offset += plan_gemm(M, it.N, it.K, bits).xs_bytes;
            sm[distinct++] = SmoothItem{it.x, it.s, xs, it.K, it.act_scale};
        }
        const int form = kernel == kSplitKernel ? 1 : kernel == kWideWhole ? 2 : 0;
        GemmBatch &bt = batch[form];
        sizes[form][bt.count] = LayerSize{it.N, it.K};
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
    auto queue_wide = [&](GemmBatch &bt, const WideTiles &t) {
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
        if (int e = launch_wide(batch[2], queue_wide(batch[2], choose_wide(true, sizes[2], batch[2].count, (M + 31) / 32, bits, num_cus())))) return e;
    const MatrixLaunches plan = plan_launches(sizes[0], batch[0].count, sizes[1], batch[1].count, M, bits, num_cus());
    const int wide = batch[0].count > 0 ? queue_wide(batch[0], plan.halves) : 0;
    if (wide > 0 && !plan.together)
        if (int e = launch_wide(batch[0], wide)) return e;
    if (batch[1].count == 0) return 0;
    const SplitTile &t = *plan.split;
    const int split = queue_split(batch[1], 32 * t.pairs, 32 * t.blocks);
    if (!plan.together) {
        const SplitVariant sv = split_variant(bits, t.pairs, t.blocks);
        void *args[] = {&batch[1]};
        return launch(split, sv.fn, kWideVariants + sv.id, 512, sv.lds_bytes, args);
    }
    const WideVariant v = bits == 2 ? mixed_variant<2>(plan.halves, t.blocks) : bits == 3 ? mixed_variant<3>(plan.halves, t.blocks) : mixed_variant<4>(plan.halves, t.blocks);
    uint32_t wide_blocks = (uint32_t)wide * kXcds;
    void *args[] = {&batch[0], &batch[1], &wide_blocks};
    return launch(wide + split, v.fn, kWideVariants + kSplitVariants + v.id, v.threads, v.lds_bytes, args);
}

}  // namespace lcd
