// Clustering-side kernels that need no calibration data (gfx950): nearest-centroid assignment of
// dense fp16 weights (the state the reclassification rule of paper Sec. 3.2, Eq. 6 maintains),
// cluster sizes, and the merge of the two closest centroids (Sec. 3.3, Eq. 8).  All of them stream
// the matrix once; none is a contraction, so there is no matrix-core work here.
#include <hip/hip_runtime.h>
#include "lcd_internal.h"
#include "lcd_device.h"

namespace lcd {

constexpr int kAssignThreads = 256;
constexpr int kAssignCols = 64 * 8;      // columns of a row per pass of its wave
constexpr int kAssignAhead = 4;          // passes of loads on the way
constexpr int kAssignPasses = 8;         // most passes of a wave

__device__ __forceinline__ double half_bits_to_double(uint16_t b) { return (double)(float)__builtin_bit_cast(_Float16, b); }

// the next fp16 value in the order of the reals (bit patterns; -0 counts as 0)
__device__ __forceinline__ uint16_t half_next_up(uint16_t b)
{
    if ((b & 0x7fffu) == 0) return 0x0001u;
    return (b & 0x8000u) ? (uint16_t)(b - 1) : (uint16_t)(b + 1);
}

// ---- nearest centroid ------------------------------------------------------------------------
// With ascending centroids the nearest one is found by counting the boundaries (c_i + c_i+1)/2
// a weight lies strictly above (a weight ON a boundary stays with the lower centroid).  A boundary
// need not be an fp16 number, but "w > boundary" for an fp16 w is the same as "w >= u" with u the
// smallest fp16 number above the boundary; u is found once per row in fp64, where the boundary is
// exact.  The comparisons are integer ones on keys that are ordered as the fp16 numbers are, two
// weights per 32-bit register: a saturating subtraction of the boundary in the middle leaves "w >= u" in the sign bits,
// which are the index's top bit and choose the half of the boundaries that stays in question (one bitwise select
// per boundary): 4, 9 and 18 instructions for two weights at 4, 8 and 16 centroids, where counting over all boundaries
// in bit planes took 5, 15 and 37.  A search needs ascending boundaries; a wave that finds a descent in its row (centroids that
// do not ascend, a NaN) counts one boundary after the other, as slowly as that is.
// Bound: HBM, 3 bytes per weight (11008 x 4096, 8 centroids: 28 -> 24.9 us by events, 5.4 TB/s, in a kernel trace 27 in the mean and 24.5 at least;
// 4096 x 4096, 16 centroids, which the counting bound: 19.7 -> 14.9 us).  A wave works alone: no barrier stands between the boundaries and the first weights, and the
// boundaries, which cost as much as two passes, are found once per eight passes (with workgroups of a row each 28 us, with two passes
// per wave 30).  Rows longer than eight passes are cut into equal parts: 4096 x 11008 in rows of 22 passes leaves half
// of the wave slots empty and takes 27 us instead of 25.  The indices are stored with the default cache policy: the next step reads
// them (assign + 1.5 us, the three steps behind it - 2.5 us).
typedef short key_pair __attribute__((ext_vector_type(2)));
typedef unsigned short ukey_pair __attribute__((ext_vector_type(2)));

// Order of the fp16 numbers as 16-bit integers: the sign-magnitude pattern turned into two's complement, moved up so
// that the positive NaNs wrap round to the bottom: a NaN of either sign is below every boundary.
__device__ __forceinline__ key_pair ordered_keys(uint32_t halves)
{
    const uint32_t sign = __builtin_bit_cast(uint32_t, (key_pair)(__builtin_bit_cast(key_pair, halves) >> 15));
    const ukey_pair up = {0x3ff, 0x3ff};
    return __builtin_bit_cast(key_pair, (ukey_pair)(__builtin_bit_cast(ukey_pair, halves ^ (sign & 0x7fff7fffu)) + up));
}

__device__ __forceinline__ uint32_t key_above(key_pair limit, key_pair key)      // bits 15 and 31
{
    return __builtin_bit_cast(uint32_t, (key_pair)__builtin_elementwise_sub_sat(limit, key));
}
__device__ __forceinline__ key_pair choose(uint32_t mask, key_pair set, key_pair clear)
{
    return __builtin_bit_cast(key_pair, bfi(mask, __builtin_bit_cast(uint32_t, set), __builtin_bit_cast(uint32_t, clear)));
}

template <int NTHR, bool ASCENDING>   // NTHR: boundaries the container can have: 3, 7 or 15
__device__ __forceinline__ uint2v nearest_of_eight(const uint4v v, const key_pair *limit)
{
    constexpr int BITS = NTHR == 3 ? 2 : NTHR == 7 ? 3 : 4;
    uint32_t bit[4][BITS];   // [register][index bit], in bits 15 and 31
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const key_pair key = ordered_keys(v[j]);
        if constexpr (ASCENDING) {
            key_pair part[NTHR];       // the boundaries that are still in question; the middle one decides
#pragma unroll
            for (int i = 0; i < NTHR; ++i) part[i] = limit[i];
#pragma unroll
            for (int b = BITS - 1, half = NTHR / 2; b >= 0; --b, half /= 2) {
                bit[j][b] = key_above(part[half], key);
                const uint32_t mask = __builtin_bit_cast(uint32_t, (key_pair)(__builtin_bit_cast(key_pair, bit[j][b]) >> 15));
#pragma unroll
                for (int i = 0; i < half; ++i) part[i] = choose(mask, part[half + 1 + i], part[i]);
            }
        } else {
            uint32_t count = 0;
#pragma unroll
            for (int i = 0; i < NTHR; ++i) count += (key_above(limit[i], key) >> 15) & 0x10001u;
#pragma unroll
            for (int b = 0; b < BITS; ++b) bit[j][b] = count << (15 - b);   // bits 15 and 31 are read
        }
    }
    uint2v o;
#pragma unroll
    for (int h = 0; h < 2; ++h) {   // bytes 0..3: the halves of registers 2 h and 2 h + 1; bit 7 of a byte of a plane is the flag
        uint32_t word = 0;
#pragma unroll
        for (int b = BITS - 1; b >= 0; --b) {
            const uint32_t plane = perm(bit[2 * h + 1][b], bit[2 * h][b], 0x07050301u) >> (BITS - 1 - b);
            word = b == BITS - 1 ? plane : bfi(0x01010101u * (0x100u - (0x100u >> (BITS - 1 - b))), word, plane);   // the bits above this one's stay
        }
        o[h] = (word >> (8 - BITS)) & (0x01010101u * ((1u << BITS) - 1u));
    }
    return o;
}

template <int NTHR, bool ASCENDING>
__device__ __forceinline__ void assign_row(const uint16_t *from, uint8_t *to, int left, const key_pair *limit, uint4v *v)
{
    while (left > 0) {
#pragma unroll
        for (int u = 0; u < kAssignAhead; ++u) {
            const uint4v now = v[u];
            if (left > kAssignAhead * kAssignCols) v[u] = stream_load(reinterpret_cast<const uint4v *>(from + kAssignAhead * kAssignCols));
            if (left > 0) *reinterpret_cast<uint2v *>(to) = nearest_of_eight<NTHR, ASCENDING>(now, limit);
            left -= kAssignCols;
            from += kAssignCols;
            to += kAssignCols;
        }
    }
}

template <int NTHR>
__global__ void __launch_bounds__(kAssignThreads, 8) assign_kernel(const uint16_t *__restrict__ w, const uint16_t *__restrict__ codebook,
                                                                uint8_t *__restrict__ idx, int K, int ncent, int parts, int width)
{
    const int lane = threadIdx.x & 63;
    // N is a multiple of 16: every wave has a part of a row
    const uint32_t unit = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kAssignThreads / 64) + (threadIdx.x >> 6)));
    const uint32_t n = unit / (uint32_t)parts;
    const int first = (int)(unit - n * (uint32_t)parts) * width;
    const uint16_t *from = w + (size_t)n * K + first + lane * 8;
    uint8_t *to = idx + (size_t)n * K + first + lane * 8;
    const int left = min(K - first, width) - lane * 8;     // K is a multiple of 256: 8 columns are all inside or all outside
    // the first passes' weights are on the way while the boundaries are found
    uint4v v[kAssignAhead];
#pragma unroll
    for (int u = 0; u < kAssignAhead; ++u)
        if (u * kAssignCols < left) v[u] = stream_load(reinterpret_cast<const uint4v *>(from + u * kAssignCols));
    uint32_t mine = 0x7fffu;           // never passed: not in use, or NaN
    if (lane + 1 < ncent) {
        const uint16_t *row = codebook + (size_t)n * (NTHR + 1);
        const double m = 0.5 * (half_bits_to_double(row[lane]) + half_bits_to_double(row[lane + 1]));   // exact
        // rounding, also twice, is monotone: the fp16 value that m rounds to is the smallest above m, or the one below that
        uint16_t h = __builtin_bit_cast(uint16_t, (_Float16)(float)m);
        if (!(half_bits_to_double(h) > m) && (h & 0x7fffu) != 0x7c00u) h = half_next_up(h);     // (stops at infinity)
        if (h == 0) h = 0x8000u;                  // both zeros pass
        if (m == m) mine = (uint16_t)(ordered_keys(h)[0] - 1);   // one below the smallest key that passes
    }
    mine *= 0x10001u;
    key_pair limit[NTHR];
#pragma unroll
    for (int i = 0; i < NTHR; ++i) limit[i] = __builtin_bit_cast(key_pair, (uint32_t)__builtin_amdgcn_readlane((int)mine, i));
    // every lane's limit no larger than the next one's (beyond the last: itself)
    const int next = __shfl((int)mine, lane + 1 < NTHR ? lane + 1 : lane);
    if (__builtin_amdgcn_ballot_w64(lane < NTHR && (short)mine > (short)next) == 0) assign_row<NTHR, true>(from, to, left, limit, v);
    else assign_row<NTHR, false>(from, to, left, limit, v);
}

// ---- cluster sizes: one wave per row -----------------------------------------------------------------
// 32 indices of a lane become four words of one bit each (bit planes); a cluster's members among them are the set
// bits of one AND of the planes, counted by one v_bcnt per cluster: about 3 instructions per index.  Bound: HBM or
// the last-level cache, 1 byte per index (11008 x 4096, 8 clusters: 18.6 us with a private LDS counter per lane and cluster,
// now 9 us, 5 TB/s;
// 16384 x 1024, 16 clusters, whose second group is empty and is passed over: 11 -> 8 us).
// Sum over the lanes: while a lane holds several counters it hands half of them to its partner, then plain sums.
template <int HELD, int OFF>
__device__ __forceinline__ void fold_counters(uint32_t *c, int lane)
{
    if constexpr (OFF > 0) {
        if constexpr (HELD > 1) {
            const bool upper = (lane & OFF) != 0;
#pragma unroll
            for (int b = 0; b < HELD / 2; ++b) {
                const uint32_t mine = upper ? c[b + HELD / 2] : c[b], theirs = upper ? c[b] : c[b + HELD / 2];
                c[b] = mine + __shfl_xor(theirs, OFF);
            }
            fold_counters<HELD / 2, OFF / 2>(c, lane);
        } else {
            c[0] += __shfl_xor(c[0], OFF);
            fold_counters<1, OFF / 2>(c, lane);
        }
    }
}

// Up to kMergeBackwards indices a workgroup counts the rows of one of the merge kernel's workgroups, which goes through them after it.
constexpr int kCountRows = 8;    // most rows of a workgroup, one per wave
constexpr long long kMergeBackwards = 1ll << 26;
template <int SLOTS>   // 4, 8 or 16
__global__ void __launch_bounds__(kCountRows * 64) counts_kernel(const uint8_t *__restrict__ idx, uint32_t *__restrict__ counts, int K)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = (int)(blockIdx.x * (blockDim.x / 64)) + wave;     // N is a multiple of 16: every wave has a row
    const uint8_t *row = idx + (size_t)n * K;
    uint32_t c[SLOTS];
#pragma unroll
    for (int b = 0; b < SLOTS; ++b) c[b] = 0;
    constexpr int GROUPS = 2;                     // groups of 32 indices a lane has in flight
    for (int first = 0; first < K; first += GROUPS * 2048) {
        const int k0 = first + lane * 16;
        uint4v v[GROUPS][2];
#pragma unroll
        for (int g = 0; g < GROUPS; ++g)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int k = k0 + g * 2048 + h * 1024;   // 16 columns are all inside or all outside
                v[g][h] = uint4v{0u, 0u, 0u, 0u};
                if (k < K) v[g][h] = *reinterpret_cast<const uint4v *>(row + k);
                else if (first + g * 2048 < K) c[0] -= 16;   // 16 zeros that are not there
            }
#pragma unroll
        for (int g = 0; g < GROUPS; ++g) {
            if (first + g * 2048 >= K) break;
            uint32_t p[4] = {0, 0, 0, 0};
#pragma unroll
            for (int d = 0; d < 8; ++d) {         // word d's bit j of every byte to bit d of every byte of plane j
                const uint32_t word = v[g][d >> 2][d & 3];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t moved = d >= j ? word << (d >= j ? d - j : 0) : word >> (d >= j ? 0 : j - d);
                    p[j] |= moved & (0x01010101u << d);
                }
            }
#pragma unroll
            for (int b = 0; b < SLOTS; ++b) {
                const uint32_t low = ((b & 1) ? p[0] : ~p[0]) & ((b & 2) ? p[1] : ~p[1]);
                const uint32_t high = ((b & 4) ? p[2] : ~p[2]) & ((b & 8) ? p[3] : ~p[3]);
                c[b] += __builtin_popcount(low & high);
            }
        }
    }
    fold_counters<SLOTS, 32>(c, lane);
    // which counter a lane ended with: its top bits
    constexpr int LOG = SLOTS == 4 ? 2 : SLOTS == 8 ? 3 : 4;
    if ((lane & ((64 >> LOG) - 1)) == 0) counts[(size_t)n * SLOTS + (lane >> (6 - LOG))] = c[0];
}

// ---- merge ---------------------------------------------------------------------------------------
// The pair with the smallest gap (gaps are exact in fp64; the lowest pair on equal gaps) becomes the
// mean of the two weighted by their cluster sizes, correctly rounded to fp16 (ties to even).  A finite
// fp16 number is an integer multiple of 2^-24 below 2^41 in magnitude and a cluster size is below 2^32,
// so the mean is the ratio of two integers, num / den with |num| < 2^75 and den < 2^34, and "which of
// two neighbouring fp16 numbers is nearer" is an integer comparison: no rounding happens anywhere.
struct U128 { uint64_t hi, lo; };
__device__ __forceinline__ U128 mul_64x64(uint64_t a, uint64_t b) { return U128{__umul64hi(a, b), a * b}; }
__device__ __forceinline__ U128 add128(U128 a, U128 b) { const uint64_t lo = a.lo + b.lo; return U128{a.hi + b.hi + (lo < a.lo ? 1u : 0u), lo}; }
__device__ __forceinline__ U128 sub128(U128 a, U128 b) { return U128{a.hi - b.hi - (a.lo < b.lo ? 1u : 0u), a.lo - b.lo}; }   // a >= b
__device__ __forceinline__ int cmp128(U128 a, U128 b) { return a.hi != b.hi ? (a.hi < b.hi ? -1 : 1) : (a.lo != b.lo ? (a.lo < b.lo ? -1 : 1) : 0); }

// magnitude of a finite fp16 bit pattern in units of 2^-24 (monotone in the 15-bit pattern)
__device__ __forceinline__ uint64_t half_units(uint32_t h15)
{
    const uint32_t e = h15 >> 10, f = h15 & 1023u;
    return e == 0 ? (uint64_t)f : (uint64_t)(1024u + f) << (e - 1);
}

// fp16 bit pattern nearest to (na * a + nb * b) / (na + nb), ties to even; (a + b) / 2 if na = nb = 0
__device__ uint16_t weighted_mean_half(uint16_t a, uint16_t b, uint32_t na, uint32_t nb)
{
    if (na == 0 && nb == 0) na = nb = 1;
    const U128 pa = mul_64x64(half_units(a & 0x7fffu), na), pb = mul_64x64(half_units(b & 0x7fffu), nb);
    const bool sa = (a & 0x8000u) != 0, sb = (b & 0x8000u) != 0;
    U128 num;
    bool neg;
    if (sa == sb) { num = add128(pa, pb); neg = sa; }
    else if (cmp128(pa, pb) >= 0) { num = sub128(pa, pb); neg = sa; }
    else { num = sub128(pb, pa); neg = sb; }
    const uint64_t den = (uint64_t)na + nb;
    // largest pattern h with units(h) * den <= num (the mean lies between the two centroids: h <= 0x7bff): the quotient in
    // binary32 is off by less than 2^-20 of itself, so rounded to fp16 it is that pattern or the next one; one more on
    // either side is tried
    const float quotient = ((float)num.hi * 0x1p64f + (float)num.lo) * 0x1p-24f * __builtin_amdgcn_rcpf((float)den);
    uint32_t h = __builtin_bit_cast(uint16_t, (_Float16)quotient) + 1u;
    if (h > 0x7bffu) h = 0x7bffu;
#pragma unroll 1
    for (int it = 0; it < 3 && cmp128(mul_64x64(half_units(h), den), num) > 0; ++it) --h;   // units(0) is 0: stops there
    if (h < 0x7bffu) {   // nearer of h and h + 1: 2 * num against (units(h) + units(h + 1)) * den
        const U128 twice = add128(num, num);
        const int c = cmp128(twice, mul_64x64(half_units(h) + half_units(h + 1), den));
        if (c > 0 || (c == 0 && (h & 1u))) ++h;
    }
    if (num.hi == 0 && num.lo == 0) neg = false;   // a mean of exactly zero is +0; a negative one that rounds to zero keeps its sign
    return (uint16_t)(h | (neg ? 0x8000u : 0u));
}

// Merge and re-numbering, one workgroup per kMergeRows rows.  One lane per row finds the pair; the
// re-numbering (idx' = idx - (idx > a), four indices per 32-bit operation) needs nothing else, so the weighted mean, a long
// serial chain for a few lanes of the first wave, comes after that wave's share of it and hides behind the other waves and
// workgroups.  Bound: HBM, 2 bytes per index (11008 x 4096: pair and mean in a launch of their own, one thread per row,
// 6.4 + 13.3 us; in one 16.1 us).  The sizes have usually just been counted: workgroups go round-robin over the XCDs, each with its own L2, so a
// workgroup takes the rows of the counting workgroup of the same XCD, and the last rows first, which that L2 still holds:
// 16.1 -> 13.8 us.  (A row order per XCD in the assignment, the counting and the packing too, each the other way round than the
// one before it, gained nothing there: what a kernel has written is not found again.)
// Beyond 2^26 indices the last-level cache no longer holds what the round reads and writes, and the other way round costs: a whole round, forwards / backwards:
// 16384 x 2048 47.0 / 44.8 us, 11008 x 4096 58.8 / 57.1, 8192 x 7168 (4 bits) 82.3 / 81.4, 8192 x 8192 80.6 / 80.7, 16384 x 8192 165.3 / 168.4.
constexpr int kMergeRows = 8;    // N is a multiple of 16
static_assert(kCountRows == kMergeRows, "a workgroup's rows were counted on its XCD");
template <int SLOTS>   // 4, 8 or 16
__global__ void __launch_bounds__(256) merge_kernel(const uint16_t *cb_in, const uint32_t *counts, const uint8_t *idx,
                                                    uint16_t *cb_out, uint8_t *out, uint8_t *merged, int K, int ncent, uint32_t rounds)
{
    __shared__ uint32_t pair[kMergeRows];
    const uint32_t group = blockIdx.x < rounds * kXcds ? (rounds - 1 - blockIdx.x / kXcds) * kXcds + blockIdx.x % kXcds : blockIdx.x;
    const int first = (int)group * kMergeRows;
    // the rows of a workgroup are contiguous: 16 indices per thread and step, AHEAD steps on the way (the first ones
    // while the pairs are found)
    constexpr int AHEAD = 4;
    const int pieces = K / 16, steps = (kMergeRows * pieces + 255 - (int)threadIdx.x) / 256;
    const uint4v *src = reinterpret_cast<const uint4v *>(idx + (size_t)first * K) + threadIdx.x;
    uint4v *dst = reinterpret_cast<uint4v *>(out + (size_t)first * K) + threadIdx.x;
    uint4v v[AHEAD];
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
        if (u < steps) v[u] = *(src + (size_t)u * 256);
    const bool decides = threadIdx.x < kMergeRows;
    const int n = first + (int)threadIdx.x;                     // a deciding lane's row
    uint16_t cb[SLOTS];
    uint32_t sizes[SLOTS];
    int a = 0;
    if (decides) {
#pragma unroll
        for (int i = 0; i < SLOTS / 4; ++i) {                   // the whole row at once
            const uint2v c = *reinterpret_cast<const uint2v *>(cb_in + (size_t)n * SLOTS + 4 * i);
            const uint4v m = *reinterpret_cast<const uint4v *>(counts + (size_t)n * SLOTS + 4 * i);
#pragma unroll
            for (int e = 0; e < 4; ++e) { cb[4 * i + e] = (uint16_t)(c[e >> 1] >> (16 * (e & 1))); sizes[4 * i + e] = m[e]; }
        }
        double best = half_bits_to_double(cb[1]) - half_bits_to_double(cb[0]);
#pragma unroll
        for (int i = 1; i + 1 < SLOTS; ++i) {
            const double g = half_bits_to_double(cb[i + 1]) - half_bits_to_double(cb[i]);
            if (i + 1 < ncent && g < best) { best = g; a = i; }
        }
        pair[threadIdx.x] = (uint32_t)a;
        merged[n] = (uint8_t)a;
    }
    __syncthreads();
    const int rows_per_step = 256 / pieces, rest = 256 - rows_per_step * pieces;   // uniform
    int row = (int)threadIdx.x / pieces, at = (int)threadIdx.x - row * pieces;
    for (int s0 = 0; s0 < steps; s0 += AHEAD) {
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (s0 + u >= steps) break;
            const uint32_t bias = (127u - pair[row]) * 0x01010101u;     // byte + bias has bit 7 set iff byte > a (bytes < 16)
#pragma unroll
            for (int d = 0; d < 4; ++d) v[u][d] -= ((v[u][d] + bias) >> 7) & 0x01010101u;
            dst[(size_t)(s0 + u) * 256] = v[u];
            if (s0 + u + AHEAD < steps) v[u] = *(src + (size_t)(s0 + u + AHEAD) * 256);
            row += rows_per_step;
            at += rest;
            if (at >= pieces) { at -= pieces; ++row; }
        }
    }
    if (decides) {
        uint16_t ca = 0, cc = 0;
        uint32_t na = 0, nb = 0;
#pragma unroll
        for (int i = 0; i + 1 < SLOTS; ++i)
            if (i == a) { ca = cb[i]; cc = cb[i + 1]; na = sizes[i]; nb = sizes[i + 1]; }
        const uint16_t nc = weighted_mean_half(ca, cc, na, nb);
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            uint16_t v = 0;
            if (i < a) v = cb[i];
            else if (i == a) v = nc;
            else if (i < ncent - 1) v = cb[i + 1 < SLOTS ? i + 1 : i];
            cb_out[(size_t)n * SLOTS + i] = v;
        }
    }
}

int launch_assign(const uint16_t *w, const uint16_t *codebook, int ncent, int N, int K, int bits, uint8_t *idx, void *stream)
{
    const int passes = (K + kAssignCols - 1) / kAssignCols, parts = (passes + kAssignPasses - 1) / kAssignPasses;
    const int width = (passes + parts - 1) / parts * kAssignCols;
    const dim3 grid((unsigned)(N / 4 * parts)), block(kAssignThreads);
    if (bits == 2) hipLaunchKernelGGL(assign_kernel<3>, grid, block, 0, (hipStream_t)stream, w, codebook, idx, K, ncent, parts, width);
    else if (bits == 3) hipLaunchKernelGGL(assign_kernel<7>, grid, block, 0, (hipStream_t)stream, w, codebook, idx, K, ncent, parts, width);
    else hipLaunchKernelGGL(assign_kernel<15>, grid, block, 0, (hipStream_t)stream, w, codebook, idx, K, ncent, parts, width);
    return (int)hipGetLastError();
}

int launch_counts(const uint8_t *idx, int N, int K, int bits, uint32_t *counts, void *stream)
{
    const int rows = (long long)N * K <= kMergeBackwards ? kCountRows : 4;
    const dim3 grid((unsigned)(N / rows)), block(rows * 64);
    if (bits == 2) hipLaunchKernelGGL(counts_kernel<4>, grid, block, 0, (hipStream_t)stream, idx, counts, K);
    else if (bits == 3) hipLaunchKernelGGL(counts_kernel<8>, grid, block, 0, (hipStream_t)stream, idx, counts, K);
    else hipLaunchKernelGGL(counts_kernel<16>, grid, block, 0, (hipStream_t)stream, idx, counts, K);
    return (int)hipGetLastError();
}

int launch_merge(const uint16_t *cb_in, const uint32_t *counts, const uint8_t *idx_in, int ncent, int N, int K, int bits,
                 uint16_t *cb_out, uint8_t *idx_out, uint8_t *merged, void *stream)
{
    const dim3 grid((unsigned)(N / kMergeRows)), block(256);
    const uint32_t rounds = (long long)N * K <= kMergeBackwards ? grid.x / kXcds : 0;
    if (bits == 2) hipLaunchKernelGGL(merge_kernel<4>, grid, block, 0, (hipStream_t)stream, cb_in, counts, idx_in, cb_out, idx_out, merged, K, ncent, rounds);
    else if (bits == 3) hipLaunchKernelGGL(merge_kernel<8>, grid, block, 0, (hipStream_t)stream, cb_in, counts, idx_in, cb_out, idx_out, merged, K, ncent, rounds);
    else hipLaunchKernelGGL(merge_kernel<16>, grid, block, 0, (hipStream_t)stream, cb_in, counts, idx_in, cb_out, idx_out, merged, K, ncent, rounds);
    return (int)hipGetLastError();
}

}  // namespace lcd
