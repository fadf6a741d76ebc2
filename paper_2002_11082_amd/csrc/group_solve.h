// Internal header of libogq: level solves of several buckets side by side in one wavefront, each by its own group of lanes.
// Included by the kernels that hold several grouped buckets in LDS: row_kernels.h and pool_kernels.h.  Compile with -ffp-contract=off.
#ifndef OGQ_GROUP_SOLVE_H
#define OGQ_GROUP_SOLVE_H

#include "rounding_kernels.h"

namespace ogq {

// Per level: what OrqLds keeps; rank = 0: not picked by rank.
struct alignas(16) GroupLevel {
    double sum_lt, sum_le;
    float value;
    uint16_t count_lt, count_le;
    uint32_t rank;
};
static_assert(sizeof(GroupLevel) == 32, "addressed by shifts");

// Bins of a bucket, HALF per sign, monotone in the value: the bin of a magnitude grows like the logarithm of
// y = (magnitude + unit) / (largest + unit), so the bins are linear below `unit` and logarithmic above, and end at the bucket's
// largest magnitude.  With unit = mean magnitude / 32 the bin of a level of a bucket of 4096 with 1024 bins holds 8 elements of Gaussian,
// 6.5 of Student-t and 4 of two-scale values, and more than 16 in 2 to 4 % of the cases; 16 binades with 32 bins each (value_bin) hold
// 16, 10 and 4, and more than 16 in 42, 21 and 4 %.  The bins only say where an element is looked for, so neither the mean
// (that of a sample) nor the rounding in here touches a result; but every use must round alike.
struct ScaledBins {
    float scale, offset;  // y = magnitude * scale + offset
    uint32_t factor;      // bins per unit in the last place of y, times 2^32
};

template <int HALF>
__device__ __forceinline__ ScaledBins scaled_bins(float mean_magnitude, uint32_t mag_max)
{
    const float largest = __uint_as_float(mag_max);
    const float unit = fmaxf(mean_magnitude, largest * 0x1p-12f) * 0x1p-5f;  // at most 17 binades above `unit`
    ScaledBins b;
    b.scale = fminf(__builtin_amdgcn_rcpf(unit + largest), 0x1.fffffep127f);
    b.offset = fminf(unit * b.scale, 1.0f);  // (infinities: 1)
    const uint32_t range = 0x3F800000u - __float_as_uint(b.offset);
    b.factor = (uint32_t)fminf((float)HALF * 0x1p32f * __builtin_amdgcn_rcpf((float)range + 1.0f), 0x1.fffffep31f);
    return b;
}

// (y's bits - offset's bits) * factor; the minimum: rounding near the largest, NaN.
template <int HALF>
__device__ __forceinline__ uint32_t magnitude_bin(float value, const ScaledBins& b)
{
    const uint32_t y = __float_as_uint(__builtin_fmaf(__builtin_fabsf(value), b.scale, b.offset));
    return umin32(__umulhi(y - __float_as_uint(b.offset), b.factor), (uint32_t)(HALF - 1));
}

// Bin of a value (with -0 already turned into +0) counted from the middle: -HALF .. HALF - 1.
template <int HALF>
__device__ __forceinline__ int32_t signed_bin(float canonical, const ScaledBins& b)
{
    return (int32_t)magnitude_bin<HALF>(canonical, b) ^ ((int32_t)__float_as_uint(canonical) >> 31);
}

// The same for many values: the subtraction goes into the product, one multiply-add, with two registers more; they must not live through the solves
// (orq_rows_kernel<16, 2> would have 97 registers where five wavefronts per SIMD allow 96: four levels, two sweeps, 16383 buckets of 128 14.2 and 15.6 us).
__device__ __forceinline__ uint64_t bin_origin(const ScaledBins& b)
{
    uint64_t origin = 0u - (uint64_t)__float_as_uint(b.offset) * b.factor;
    asm("" : "+v"(origin));  // (known, it is turned back into a subtraction and a wider product)
    return origin;
}

template <int HALF>
__device__ __forceinline__ int32_t signed_bin(float canonical, const ScaledBins& b, uint64_t origin)
{
    const uint32_t y = __float_as_uint(__builtin_fmaf(__builtin_fabsf(canonical), b.scale, b.offset));
    const uint32_t bin = umin32((uint32_t)(((uint64_t)y * b.factor + origin) >> 32), (uint32_t)(HALF - 1));
    return (int32_t)bin ^ ((int32_t)__float_as_uint(canonical) >> 31);
}

// Grouping.  A bin's counter begins as the LDS address of its entry of `bin_start` in the upper half and that of the grouped values in the
// lower one, and counts in bytes.  So what the returning add hands an element holds both addresses that the scatter needs, already added up: a
// shift for the start, a 16-bit addition for the place: two vector instructions per element where packing position and counter, and two additions
// to each half, took five (25.6 M values in buckets of 2048, four levels, 45.9 -> 44.4 us; 143.7 M in buckets of 4096, eight, 293 -> 289).
__device__ __forceinline__ uint32_t counter_start(uint32_t starts, uint32_t grouped, uint32_t bin) { return (starts << 16 | grouped) + (bin << 17); }

// Two starts of 16 bits, whatever lies above.
__device__ __forceinline__ uint32_t two_starts(uint32_t start, uint32_t next) { return __builtin_amdgcn_perm(next, start, 0x05040100u); }

// LDS address of the element's place in the grouped values, from what its counter returned.
__device__ __forceinline__ uint32_t place_in_bin(uint32_t slot)
{
    return (uint16_t)(*(const LdsHalf*)(uintptr_t)(slot >> 16) + (uint16_t)slot);
}

// A bucket in LDS as one lane of its group sees it.
struct GroupBucket {
    const char* grouped;        // fp32 bit patterns by bin
    const uint16_t* bin_start;  // byte offset of every bin's first position in `grouped`; points at the middle bin's
    const double* prefix;       // sum of the bucket's elements before every BLOCK-th position of `grouped`
    GroupLevel* level;
    unsigned long long* limb;   // workspace of exact_floor_t, the same for all groups
    ScaledBins bins;
    uint32_t origin, len;       // the bucket's first position in `grouped`, its elements
    double bound;               // sum_error_bound (floor_t_from_sums)
};

__device__ __forceinline__ float grouped_value(const char* at) { return __uint_as_float(*reinterpret_cast<const uint32_t*>(at)) + 0.0f; }

// Ascending sort of K keys per lane over every group of G lanes: element K * (lane in the group) + register.  The first step
// of a merge of runs of N elements pairs e with e ^ (2 N - 1), the others e with e ^ J (see wave_sort_merge).
template <int J, int K>
__device__ __forceinline__ void group_sort_steps(uint32_t (&x)[K], uint32_t lane)
{
    if constexpr (J >= K) {
        const uint32_t bound = upper_lanes<J / K>(lane);
#pragma unroll
        for (int r = 0; r < K; ++r) x[r] = smaller_or_larger(x[r], lane_xor<J / K>(x[r], lane), bound);
    } else if constexpr (J >= 1) {
#pragma unroll
        for (int r = 0; r < K; ++r)
            if ((r & J) == 0) sort_pair(x[r], x[r | J]);
    }
    if constexpr (J > 1) group_sort_steps<J / 2, K>(x, lane);
}

template <int G, int K, int N = 1>
__device__ __forceinline__ void group_sort(uint32_t (&x)[K], uint32_t lane)
{
    if constexpr (2 * N <= K * G) {
        if constexpr (2 * N <= K) {
#pragma unroll
            for (int r = 0; r < K; ++r)
                if (r < (r ^ (2 * N - 1))) sort_pair(x[r], x[r ^ (2 * N - 1)]);
        } else {
            const uint32_t bound = upper_lanes<N / K>(lane);
            uint32_t y[K];
#pragma unroll
            for (int r = 0; r < K; ++r) y[r] = lane_reverse<N / K>(x[K - 1 - r], lane);
#pragma unroll
            for (int r = 0; r < K; ++r) x[r] = smaller_or_larger(x[r], y[r], bound);
        }
        if constexpr (N > 1) group_sort_steps<N / 2, K>(x, lane);
        group_sort<G, K, 2 * N>(x, lane);
    }
}

// Largest key of the group, in all its lanes.
template <int G>
__device__ __forceinline__ uint32_t group_max(uint32_t x)
{
    x = umax32(x, dpp_u32<kDppXor1>(x));
    x = umax32(x, dpp_u32<kDppXor2>(x));
    x = umax32(x, dpp_u32<kDppHalfMirror>(x));
    if constexpr (G == 16) x = umax32(x, dpp_u32<kDppMirror>(x));
    return x;
}

// Lanes of this lane's group of G for which the condition holds.
template <int G>
__device__ __forceinline__ uint32_t group_count(bool condition, uint32_t lane)
{
    return (uint32_t)__popc((uint32_t)(__ballot(condition) >> (lane & (64u - (uint32_t)G))) & ((1u << G) - 1u));
}

// x[index % K].  By masks: a choice between two elements of an array becomes a load from a chosen address before the array is
// split into registers, and then it stays in scratch memory, or is moved to LDS with the lane's place computed from the dispatch
// packet in host memory, which every wavefront waits 13 us for.
template <int K>
__device__ __forceinline__ uint32_t picked_register(const uint32_t (&x)[K], uint32_t index)
{
    static_assert(K == 1 || K == 2 || K == 4, "");
    if constexpr (K == 1) return x[0];
    const uint32_t odd = 0u - (index & 1u);
    const uint32_t low = (x[0] & ~odd) | (x[K > 1 ? 1 : 0] & odd);
    if constexpr (K == 2) return low;
    const uint32_t high = (x[K > 2 ? 2 : 0] & ~odd) | (x[K > 2 ? 3 : 0] & odd), upper = 0u - (index >> 1 & 1u);
    return (low & ~upper) | (high & upper);
}

// An element picked by rank, the same in all lanes of a group; counts and sum are those of its bin.
struct GroupPicked {
    float value;
    uint32_t count_lt, count_le;
    double part;  // this lane's share of the sum of the smaller elements
};

// The element of index `index` (0-based) among the n (at most WITHIN K, WITHIN <= G) values at `at`.
template <int G, int K, bool SUMS, int WITHIN = G>
__device__ __forceinline__ GroupPicked group_pick_sorted(const char* at, uint32_t n, uint32_t index, uint32_t lane)
{
    const uint32_t i = lane & (uint32_t)(G - 1);
    float value[K];
    uint32_t mine[K], x[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        // (a lane past the n reads whatever of the LDS record follows and drops it)
        value[k] = grouped_value(at + 4u * (i + (uint32_t)(G * k)));
        mine[k] = i + (uint32_t)(G * k) < n ? float_to_key(value[k]) : 0xFFFFFFFFu;
        x[k] = mine[k];
    }
    group_sort<WITHIN, K>(x, lane);  // (past WITHIN lanes there is only padding)
    // element `index`, handed to all lanes of the group as the largest of what they offer
    const uint32_t key = group_max<G>(i == index / (uint32_t)K ? picked_register<K>(x, index) : 0u);
    GroupPicked p{key_to_float(key), 0u, 0u, 0.0};
    if constexpr (SUMS && K == 1) {
        const bool below = mine[0] < key;
        p.part = (double)(below ? value[0] : 0.0f);
        p.count_lt = group_count<G>(below, lane);
        p.count_le = umin32(group_count<G>(mine[0] <= key, lane), n);  // (a key of all ones, a NaN, equals the padding)
    } else if constexpr (SUMS) {
        uint32_t counts = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool below = mine[k] < key;
            counts += (below ? 1u : 0u) + (mine[k] <= key ? 0x10000u : 0u);
            p.part += (double)(below ? value[k] : 0.0f);
        }
        counts = row_sum_u32<G>(counts, lane);
        p.count_lt = counts & 0xFFFFu;
        p.count_le = umin32(counts >> 16, n);
    }
    return p;
}

// The same for a crowded bin (some group's bin holds more than fits the sort).  bin = the LDS address of its first element; n = 0: no
// element is wanted.  What crowds a bin in earnest is one value that many elements share: zero in a sparse gradient, the threshold
// in a clipped one.  So the pivots are elements: a pass over the bin counts what lies below and at the pivot, and ends the search
// where the wanted index is among the equals, which the first pass does as often as the shared value is wanted.  Otherwise it
// leaves a range of keys, and the next pivot is one of G elements drawn from the bin.  Where none of them lies in the range, and at every
// fourth pass (which bounds the search whatever the elements), the range is narrowed to keys that elements have, and the pivot is its
// middle.  Bisection over the bits of the key took some 20 passes (us, bisection -> this): eight levels, two sweeps, c = 2.5, 64 buckets of
// 4096 of a mixture of scales 55 -> 17; half of the values zero, 25.6 M of them in buckets of 4096 2063 -> 148, in buckets of 256 (no
// sweeps) 426 -> 118.
template <int G, bool SUMS>
__device__ __forceinline__ GroupPicked group_pick_crowded(uint32_t bin, uint32_t n, uint32_t index, uint32_t lane)
{
    const uint32_t i = lane & (uint32_t)(G - 1);
    const LdsWord* at = (const LdsWord*)(uintptr_t)bin;
    index = umin32(index, n - 1u);  // (a search beyond the bin would not end)
    const uint32_t wanted = __float_as_uint(__uint_as_float(at[n != 0u ? index : 0u]) + 0.0f);
    const uint32_t order = wanted >> 31 != 0u ? 0xFFFFFFFFu : 0x80000000u;  // float_to_key: a bin's elements have one sign
    auto key_at = [&](uint32_t e) __attribute__((always_inline)) { return __float_as_uint(__uint_as_float(at[e]) + 0.0f) ^ order; };
    auto each = [&](uint32_t end, auto f) __attribute__((always_inline)) {
        uint32_t e = i;
#pragma unroll 1
        for (; e + 3u * (uint32_t)G < end; e += 4u * (uint32_t)G) {
            uint32_t key[4];
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k) key[k] = key_at(e + (uint32_t)G * k);
#pragma unroll
            for (int k = 0; k < 4; ++k) f(key[k]);
        }
#pragma unroll 1
        for (; e < end; e += (uint32_t)G) f(key_at(e));
    };
    GroupPicked p{0.0f, 0u, 0u, 0.0};
    uint32_t lo = 0u, hi = 0xFFFFFFFFu, pivot = wanted ^ order;
    uint32_t rest = n;  // 0 once the element is found
#pragma unroll 1
    for (uint32_t step = 1;; ++step) {
        uint32_t counts = 0u, not_above = 0u;
        double part = 0.0;
        each(rest, [&](uint32_t key) __attribute__((always_inline)) {
            const bool lt = key < pivot;
            counts += lt ? 1u : 0u;
            not_above += key <= pivot ? 1u : 0u;
            if constexpr (SUMS) part += (double)__uint_as_float(lt ? key ^ order : 0u);
        });
        counts = row_sum_u32<G>(counts | not_above << 16, lane);
        const uint32_t below = counts & 0xFFFFu;
        not_above = counts >> 16;
        if (rest != 0u && below <= index && index < not_above) {
            p = GroupPicked{__uint_as_float(pivot ^ order), below, not_above, part};
            rest = 0u;
        }
        if (__ballot(rest != 0u) == 0) break;
        if (index < below) hi = pivot - 1u;
        else lo = pivot + 1u;
        const uint32_t sample = key_at(__umulhi((i + (uint32_t)G * step) * 0x9E3779B1u, n));
        const bool inside = lo <= sample && sample <= hi;
        const uint32_t first = group_max<G>(inside ? (uint32_t)G - i : 0u);  // (the first lane whose element does)
        const bool drawn = first != 0u && (step & 3u) != 0u;
        pivot = group_max<G>((uint32_t)G - i == first ? sample : 0u);
        if (__ballot(rest != 0u && !drawn) != 0) {
            uint32_t smallest = 0xFFFFFFFFu, largest = 0u;
            each(drawn ? 0u : rest, [&](uint32_t key) __attribute__((always_inline)) {
                const bool in_range = lo <= key && key <= hi;
                smallest = in_range ? umin32(smallest, key) : smallest;
                largest = in_range ? umax32(largest, key) : largest;
            });
            smallest = row_min_u32<G>(smallest, lane);
            largest = row_max_u32<G>(largest, lane);
            lo = drawn ? lo : smallest;
            hi = drawn ? hi : largest;
            pivot = drawn ? pivot : lo + ((hi - lo) >> 1);
        }
    }
    return p;
}

// Out of line for the level solves: inlined into their loops it cost solves that never need it 0.5 to 1 %.
template <int G>
static __device__ __attribute__((noinline)) GroupPicked group_pick_crowded_with_sums(uint32_t bin, uint32_t n, uint32_t index, uint32_t lane)
{
    return group_pick_crowded<G, true>(bin, n, index, lane);
}

// floor(T) of one group's bucket in exact arithmetic (see exact_floor_t), by the whole wavefront; elements = the LDS address of the
// bucket's first one.
__device__ __forceinline__ uint32_t exact_floor_t_elements(unsigned long long* limb, uint32_t elements, uint32_t len, uint32_t lane, float L,
                                                           float R, uint32_t count_in, uint32_t guess)
{
    return exact_floor_t(limb, lane, L, R, count_in, guess, [&](auto add) {
        for (uint32_t i = lane; i < len; i += kWave) add(__uint_as_float(((const LdsWord*)(uintptr_t)elements)[i]) + 0.0f);
    });
}

static __device__ __attribute__((noinline)) uint32_t exact_floor_t_group(unsigned long long* limb, uint32_t elements, uint32_t len,
                                                                         uint32_t lane, float L, float R, uint32_t count_in,
                                                                         uint32_t guess)
{
    return exact_floor_t_elements(limb, elements, len, lane, L, R, count_in, guess);
}

// Truncation that takes negative values and NaN to 0 (v_cvt_u32_f64 saturates; the conversion of the language does not).
__device__ __forceinline__ uint32_t truncated_u32(double x)
{
    uint32_t r;
    asm("v_cvt_u32_f64_e32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// The same value, of which the compiler does not know it: what a rare branch needs of the LDS it reads again, instead of registers
// that hold it through the pick (the kernels have none to spare).
__device__ __forceinline__ uint32_t read_again(uint32_t entry)
{
    asm("" : "+v"(entry));
    return entry;
}

// One level solve per group of G lanes, run by a whole wavefront: level k between the levels l and r of the group's bucket (see
// orq_solve_one), entry = k | l << 4 | r << 8, 0 for a group with nothing to do.  SUMS = false: one interior level,
// whose solve reads the bucket's total alone.  Shape: HALF (signed_bin), BLOCK (positions per entry of the
// prefix), END_OF_BUCKET (the entry behind a bucket's last bin is not its end) and LEAF (a function of its own, which calls none).
// Returns whether a level has moved (LEAF alone; else whether one was solved).
//
// The bin of a rank needs no search: the element at that position of the grouped bucket is in it.  The element of the rank is then
// found by sorting the bin.
template <int G, bool SUMS, class Shape>
__device__ __forceinline__ bool group_solve(const GroupBucket& b, uint32_t entry, uint32_t lane)
{
    constexpr uint32_t BLOCK = Shape::BLOCK, LANES = (uint32_t)G;
    static_assert(!SUMS || BLOCK % LANES == 0, "the elements in front of a bin are read G at a time");
    const uint32_t i = lane & (LANES - 1u);
    const uint32_t k = entry & 15u;
    const GroupLevel left = b.level[(entry >> 4) & 15u], right = b.level[entry >> 8];
    const uint32_t last_rank = b.level[k].rank;
    const float L = left.value, R = right.value;
    const bool ordered = L < R;
    // S = sum_{L<=v<=R} (v - L),  T = S / (R - L),  level = element of rank #{v<=R} - floor(T)
    const uint32_t count_in = (uint32_t)right.count_le - left.count_lt;
    const double width = (double)R - (double)L;
    const double Ssum = __builtin_fma(-(double)L, (double)count_in, right.sum_le - left.sum_lt);
    // floor_t_from_sums without branches; m is not used when L == R
    uint32_t m = truncated_u32(Ssum * __builtin_amdgcn_rcp(width));
    const double rest = __builtin_fma(-(double)m, width, Ssum);
    const bool over = rest >= width, under = rest < 0.0 && m > 0u;
    m = m + (over ? 1u : 0u) - (under ? 1u : 0u);
    const double settled = rest - (over ? width : under ? -width : 0.0);
    const bool undecided = ordered && b.bound != 0.0 && !(settled > b.bound && width - settled > b.bound);
    for (uint64_t todo = __ballot(undecided && i == 0u); todo != 0; todo &= todo - 1u) {  // (rare) one group after the other
        const uint32_t of = (uint32_t)__builtin_ctzll(todo);
        const uint32_t elements = (uint32_t)(uintptr_t)((const LdsWord*)b.grouped) + 4u * b.origin;
        const uint32_t first = __builtin_amdgcn_readlane(elements, of), len = __builtin_amdgcn_readlane(b.len, of);
        const uint32_t in = __builtin_amdgcn_readlane(count_in, of), guess = __builtin_amdgcn_readlane(m, of);
        const uint32_t exact = Shape::LEAF ? exact_floor_t_elements(b.limb, first, len, lane, readlane_f32(L, of), readlane_f32(R, of), in, guess)
                                           : exact_floor_t_group(b.limb, first, len, lane, readlane_f32(L, of), readlane_f32(R, of), in, guess);
        m = lane / LANES == of / LANES ? exact : m;
    }
    const uint32_t rank = umin32(umax32(__builtin_elementwise_sub_sat((uint32_t)right.count_le, m), 1u), b.len);
    const bool same = entry == 0u || (ordered && rank == last_rank);  // same element as last time
    if (__ballot(!same) == 0) return false;

    const uint32_t at = b.origin + (rank > 0u ? rank - 1u : 0u);  // (rank 0: an empty bucket)
    const int32_t bin = signed_bin<Shape::HALF>(grouped_value(b.grouped + 4u * at), b.bins);
    const uint32_t first = (uint32_t)b.bin_start[bin] >> 2;
    uint32_t last = (uint32_t)b.bin_start[bin + 1] >> 2;
    if constexpr (Shape::END_OF_BUCKET) last = umin32(last, b.origin + b.len);
    double before = 0.0, part = 0.0;
    if constexpr (SUMS) {
        // the sum of everything before the bin: the prefix of its block, and the block's positions in front of it
        before = b.prefix[first / BLOCK];
        const uint32_t in_front = first & (BLOCK - 1u);
        const char* block = b.grouped + 4u * (first - in_front + i);
#pragma unroll
        for (uint32_t c = 0; c < BLOCK / LANES; ++c) {
            const float x = __uint_as_float(*reinterpret_cast<const uint32_t*>(block + 4u * LANES * c));
            part += (double)(i + LANES * c < in_front ? x : 0.0f);
        }
    }
    GroupPicked p;
    const uint32_t n = same || !ordered ? 0u : last - first;  // (0: nothing is picked, and no other group waits for this one)
    const char* keys = b.grouped + 4u * first;
    if (__ballot(n > 8u) == 0) p = group_pick_sorted<G, 1, SUMS, 8>(keys, n, at - first, lane);
    else if (__ballot(n > LANES) == 0) p = group_pick_sorted<G, 1, SUMS>(keys, n, at - first, lane);
    else if (__ballot(n > 2u * LANES) == 0) p = group_pick_sorted<G, 2, SUMS>(keys, n, at - first, lane);
    else if (__ballot(n > 4u * LANES) == 0) p = group_pick_sorted<G, 4, SUMS>(keys, n, at - first, lane);
    else {
        // Is it one of the elements that this level, or a level beside it, has been found equal to?
        bool equal = false;
        if constexpr (SUMS) {
            const uint32_t again = read_again(entry);
#pragma unroll
            for (uint32_t shift = 0; shift <= 8u; shift += 4u) {
                const uint32_t level = (again >> shift) & 15u;
                const GroupLevel x = b.level[level];
                const double rest = x.sum_lt - before;  // (not of infinities)
                if (x.rank != 0u && x.count_lt < rank && rank <= x.count_le && rest == rest) {
                    equal = true;
                    p = GroupPicked{x.value, x.count_lt - (first - b.origin), x.count_le - (first - b.origin), 0.0};
                    part = i == 0u ? rest : 0.0;
                }
            }
        }
        const uint32_t elements = (uint32_t)(uintptr_t)(const LdsWord*)keys, search = equal ? 0u : n;
        const GroupPicked found = SUMS && !Shape::LEAF ? group_pick_crowded_with_sums<G>(elements, search, at - first, lane)
                                                       : group_pick_crowded<G, SUMS>(elements, search, at - first, lane);
        if (!equal) p = found;
    }
    GroupLevel now{0.0, 0.0, p.value, 0, 0, rank};
    if constexpr (SUMS) {
        now.sum_lt = before + row_sum_f64<G>(part + p.part, lane);
        now.sum_le = __builtin_fma((double)(p.count_le - p.count_lt), (double)p.value, now.sum_lt);
        const uint32_t in_front = first - b.origin;
        now.count_lt = (uint16_t)(in_front + p.count_lt);
        now.count_le = (uint16_t)(in_front + p.count_le);
    }
    const bool copy_left = !ordered || p.value < L;  // the level coincides with the left end
    if (__ballot(copy_left) != 0) {                  // (rare: nothing to select otherwise)
        now.value = copy_left ? L : now.value;
        now.rank = copy_left ? 0u : now.rank;
        if constexpr (SUMS) {
            const uint32_t again = read_again(entry);
            const GroupLevel left = b.level[(again >> 4) & 15u], right = b.level[again >> 8];
            now.count_lt = copy_left ? left.count_lt : now.count_lt;
            now.count_le = copy_left ? (ordered ? left.count_le : right.count_le) : now.count_le;
            now.sum_lt = copy_left ? left.sum_lt : now.sum_lt;
            now.sum_le = copy_left ? (ordered ? left.sum_le : right.sum_le) : now.sum_le;
        }
    }
    bool moved = true;
    if constexpr (Shape::LEAF) moved = __ballot(!same && __float_as_uint(now.value) != __float_as_uint(b.level[read_again(entry) & 15u].value)) != 0;
    if (i == 0u && !same) b.level[k] = now;
    wave_lds_sync();
    return moved;
}

// ----------------------------------------------------------------------------------------------
// The same solve as a straight line, by groups of 16 lanes, for a wavefront that others wait for.  What bounds it is the number of its
// instructions (one wavefront issues one in four cycles) and its branches and trips to LDS (30 to 45 and 60 cycles each), so little is
// tested before the end.  The element is found by counting: every lane takes one of the 16 elements from the bin's first on (two of 32
// where a bin is larger) and counts those that are smaller than its own; what they hold beyond the bin is larger than everything in it.
// Returns false, and leaves the level alone, where that does not do for some active group: floor(T) not settled by its first guess, a
// bin of more than 32 elements, a value that several elements share, L == R, a bucket that is not `ordinary`; the general solve then takes the
// step.  Eight levels, two sweeps, buckets of 4096 of Student-t values: one step in 4,100 does, and a step takes 1,300 cycles; both kinds of
// picks in one line of branches took 2,000 (profiles/phase_cycles.txt).
// ----------------------------------------------------------------------------------------------
typedef __attribute__((address_space(3))) const double LdsDouble;
typedef __attribute__((address_space(3))) GroupLevel LdsLevel;

// A bucket in LDS as one lane of its group sees it; LDS addresses.  The bucket's first position is 0.
struct DirectBucket {
    uint32_t grouped, own;     // first element; the one at the lane's place in the group
    uint32_t bin_start, prefix;
    ScaledBins bins;
    uint32_t last, end;        // index of the last element; 4 times that of the last 16's first one
    uint64_t ordinary;         // lanes whose bucket has at least 32 elements and a finite sum
    double low, high;          // a rest above `low` and further than `high` from the width settles floor(T)
};

__device__ __forceinline__ DirectBucket direct_bucket(const GroupBucket& b, bool finite, uint32_t lane)
{
    DirectBucket d;
    d.grouped = (uint32_t)(uintptr_t)(const LdsWord*)b.grouped;
    d.own = d.grouped + 4u * (lane & 15u);
    d.bin_start = (uint32_t)(uintptr_t)(const LdsHalf*)b.bin_start;
    d.prefix = (uint32_t)(uintptr_t)(LdsDouble*)b.prefix;
    d.bins = b.bins;
    d.last = b.len > 0u ? b.len - 1u : 0u;
    d.end = b.len >= 32u ? 4u * (b.len - 16u) : 64u;
    d.ordinary = __ballot(finite && b.len >= 32u);
    d.low = b.bound != 0.0 ? b.bound : -0x1p-1022;  // (exact sums: 0 settles it too)
    d.high = b.bound;
    return d;
}

// How many of the 16 elements `other` of the row are smaller than this lane's `own` (finite values, no -0): a move across the row with
// a subtraction, and a shift that takes the sign, for each.  In assembly because the compiler puts a wait state into every pair.  Wait
// states: two between whatever wrote `other` and the first move.  All lanes are active.
__device__ __forceinline__ uint32_t smaller_in_row(float other, float own)
{
    uint32_t signs, d0, d1;
#define OGQ_TURN(a, b) \
    "v_sub_f32_dpp %[d0], %[other], %[own] row_ror:" a " row_mask:0xf bank_mask:0xf\n\t" \
    "v_sub_f32_dpp %[d1], %[other], %[own] row_ror:" b " row_mask:0xf bank_mask:0xf\n\t" \
    "v_alignbit_b32 %[signs], %[signs], %[d0], 31\n\t" \
    "v_alignbit_b32 %[signs], %[signs], %[d1], 31\n\t"
    asm("v_sub_f32_e32 %[signs], %[other], %[own]\n\t"
        "v_lshrrev_b32_e32 %[signs], 31, %[signs]\n\t"
        "v_sub_f32_dpp %[d0], %[other], %[own] row_ror:15 row_mask:0xf bank_mask:0xf\n\t"
        "v_alignbit_b32 %[signs], %[signs], %[d0], 31\n\t"
        OGQ_TURN("1", "2") OGQ_TURN("3", "4") OGQ_TURN("5", "6") OGQ_TURN("7", "8") OGQ_TURN("9", "10") OGQ_TURN("11", "12") OGQ_TURN("13", "14")
        "v_bcnt_u32_b32 %[signs], %[signs], 0"
        : [signs] "=&v"(signs), [d0] "=&v"(d0), [d1] "=&v"(d1)
        : [other] "v"(other), [own] "v"(own));
#undef OGQ_TURN
    return signs;
}

// The end of a direct solve, K elements per lane: picks element `at`, whose bin begins at `first` (times 4), writes the level's record.
template <int K, class Shape>
__device__ __forceinline__ bool direct_pick(const DirectBucket& b, uint32_t at, uint32_t first, uint32_t level, uint64_t settled,
                                            uint64_t active, uint32_t lane)
{
    constexpr uint32_t BLOCK = Shape::BLOCK, G = 16;
    static_assert(BLOCK % G == 0 && !Shape::END_OF_BUCKET, "the elements in front of a bin are read G at a time");
    const uint32_t i4 = 4u * (lane & (G - 1u));
    const uint32_t from = umin32(first, b.end - (K == 2 ? 4u * G : 0u));
    const LdsWord* mine = (const LdsWord*)(uintptr_t)(b.own + from);
    float own[K];
#pragma unroll
    for (int k = 0; k < K; ++k) own[k] = __uint_as_float(mine[G * k]) + 0.0f;
    // the sum of everything before `from`: the prefix of its block, and the block's positions in front of it
    const uint32_t in_front = from & (4u * BLOCK - 1u);
    const LdsWord* block = (const LdsWord*)(uintptr_t)(b.own + (from - in_front));
    const double before = *(LdsDouble*)(uintptr_t)(b.prefix + 8u * (from / (4u * BLOCK)));
    float front[BLOCK / G];
#pragma unroll
    for (uint32_t c = 0; c < BLOCK / G; ++c) front[c] = __uint_as_float(block[G * c]);
    uint32_t bits = 0;
    uint64_t found = 0, twice = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        uint32_t smaller = smaller_in_row(own[0], own[k]);
        if constexpr (K == 2) smaller += smaller_in_row(own[1], own[k]);
        const bool is_it = smaller == at - from / 4u;
        const uint64_t lanes = __ballot(is_it) & active;
        twice |= found & lanes;
        found |= lanes;
        bits |= is_it ? __float_as_uint(own[k]) : 0u;
    }
    bits |= dpp_u32<kDppXor1>(bits);
    bits |= dpp_u32<kDppXor2>(bits);
    bits |= dpp_u32<kDppHalfMirror>(bits);
    bits |= dpp_u32<kDppMirror>(bits);
    const float value = __uint_as_float(bits);
    double part = 0.0;
#pragma unroll
    for (uint32_t c = 0; c < BLOCK / G; ++c) part += (double)(i4 + 4u * G * c < in_front ? front[c] : 0.0f);
#pragma unroll
    for (int k = 0; k < K; ++k) part += (double)(own[k] < value ? own[k] : 0.0f);
    const double sum_lt = before + row_sum_f64<16>(part, lane);
    asm volatile("" ::"v"(sum_lt));  // (what it takes is read with the elements, not behind the branch)

    // one lane of every active group has found it: where several elements share a value, none or several have
    const uint64_t firsts = active & 0x0001000100010001ull;
    const uint64_t amiss = twice | (found & (found - firsts)) | (active & ~settled);
    if (__builtin_expect((amiss | (uint64_t)(uint32_t)(__popcll(found) - __popcll(firsts))) != 0, 0)) return false;

    LdsLevel* out = (LdsLevel*)(uintptr_t)level;  // (the same from all lanes of the group)
    out->sum_lt = sum_lt;
    out->sum_le = sum_lt + (double)value;
    out->value = value;
    out->count_lt = (uint16_t)at;
    out->count_le = (uint16_t)(at + 1u);
    out->rank = at + 1u;
    wave_lds_sync();
    return true;
}

// left, right, level: LDS addresses of the records (level: of one that nothing reads for the other groups); active: the lanes (whole
// groups) that solve.  SKIP: a level that every active group finds at the rank it already has is left as it is, and `changed` is set where one is
// not.
template <class Shape, bool SKIP>
__device__ __forceinline__ bool group_solve_direct(const DirectBucket& b, uint32_t left, uint32_t right, uint32_t level, uint64_t active,
                                                   uint32_t lane, bool& changed)
{
    const uint32_t last_rank = SKIP ? ((const LdsLevel*)(uintptr_t)level)->rank : 0u;
    const floatx2 of_left = *(const LdsPair*)(uintptr_t)(left + 16u), of_right = *(const LdsPair*)(uintptr_t)(right + 16u);
    const double sum_in = ((const LdsLevel*)(uintptr_t)right)->sum_le - ((const LdsLevel*)(uintptr_t)left)->sum_lt;
    const uint32_t not_above = __float_as_uint(of_right.y) >> 16;
    const double L = (double)of_left.x, width = (double)of_right.x - L;
    const double Ssum = __builtin_fma(-L, (double)(not_above - (__float_as_uint(of_left.y) & 0xFFFFu)), sum_in);
    const uint32_t m = truncated_u32(Ssum * __builtin_amdgcn_rcp(width));
    const double rest = __builtin_fma(-(double)m, width, Ssum);
    const uint64_t settled = __ballot(rest > b.low) & __ballot(width - rest > b.high) & b.ordinary;
    const uint32_t at = umin32(not_above - m - 1u, b.last);  // (in range whatever m is)
    if constexpr (SKIP) {
        if (((__ballot(at + 1u != last_rank) | ~settled) & active) == 0) return true;
        changed = true;
    }
    const float element = __uint_as_float(*(const LdsWord*)(uintptr_t)(b.grouped + 4u * at)) + 0.0f;
    const LdsHalf* bin = (const LdsHalf*)(uintptr_t)(b.bin_start + 2u * (uint32_t)signed_bin<Shape::HALF>(element, b.bins));
    const uint32_t first = bin[0], size = bin[1] - first;
    if (__builtin_expect((__ballot(size > 64u) & active) != 0, 0)) {
        if ((__ballot(size > 128u) & active) != 0) return false;
        return direct_pick<2, Shape>(b, at, first, level, settled, active, lane);
    }
    return direct_pick<1, Shape>(b, at, first, level, settled, active, lane);
}

// What a crowded bin has shown of a group's bucket: the elements before index `end` of the sorted bucket are at most `value`.
struct GroupTie {
    float value;
    uint32_t end;
};

// The element of 0-based index `index` of every group's sorted bucket (one chain), indexes in ascending order from call to call.
template <int G, class Shape>
__device__ __forceinline__ float group_element(const GroupBucket& b, uint32_t index, GroupTie& tie, uint32_t lane)
{
    const uint32_t at = b.origin + index;
    const int32_t bin = signed_bin<Shape::HALF>(grouped_value(b.grouped + 4u * at), b.bins);
    const uint32_t first = (uint32_t)b.bin_start[bin] >> 2;
    uint32_t last = (uint32_t)b.bin_start[bin + 1] >> 2;
    if constexpr (Shape::END_OF_BUCKET) last = umin32(last, b.origin + b.len);
    const uint32_t n = last - first;
    const char* keys = b.grouped + 4u * first;
    if (__ballot(n > (uint32_t)G) == 0) return group_pick_sorted<G, 1, false>(keys, n, at - first, lane).value;
    if (__ballot(n > 2u * (uint32_t)G) == 0) return group_pick_sorted<G, 2, false>(keys, n, at - first, lane).value;
    if (__ballot(n > 4u * (uint32_t)G) == 0) return group_pick_sorted<G, 4, false>(keys, n, at - first, lane).value;
    const bool known = index < tie.end;  // (no element before this one is larger than it)
    const GroupPicked p = group_pick_crowded<G, false>((uint32_t)(uintptr_t)(const LdsWord*)keys, known ? 0u : n, at - first, lane);
    if (!known) tie = GroupTie{p.value, first - b.origin + p.count_le};
    return tie.value;
}

// The greedy steps of a chain, 12 bits each; head: with the first solves of the first sweep in the steps that have room for them.
constexpr uint64_t packed_entries(const TeamGreedy& greedy, int chain, bool head)
{
    uint64_t packed = 0;
    for (int step = 0; step < greedy.steps; ++step) {
        uint64_t e = greedy.entry[chain][step];
        for (int h = 0; h < 2; ++h)
            if (head && greedy.head_step[h] == step) e = (uint64_t)(h + 1) * 0x111u + 0x0F0u;
        packed |= e << (12 * step);
    }
    return packed;
}

// All level solves of the groups' buckets, CHAINS = 1 or 2 groups per bucket (group lane / G of the wavefront is chain
// (lane / G) % CHAINS of its bucket).  One chain: Algorithm 1's order, then the sweeps.  Two chains: the schedule of
// orq_team_solve, i.e. the halves on either side of Algorithm 1's first level, and of each pair of sweeps the second two levels
// behind the first; the results are those of the serial order.
template <int G, int CHAINS, int S, class Shape>
__device__ __forceinline__ void group_solve_levels(const GroupBucket& b, uint32_t sweeps, uint32_t lane)
{
    constexpr bool SUMS = S > 3;
    constexpr uint32_t INTERIOR = S - 2;
    constexpr uint32_t kNext = 0x111u, kFirst = 0x201u;  // from a level's entry of a sweep to the next one's; that of level 1
    if constexpr (CHAINS == 1) {
        constexpr GreedyOrder order = greedy_order<S>();
        uint32_t steps = order.count + (S > 3 ? sweeps * INTERIOR : 0u);  // (one interior level: sweeps repeat it)
        uint32_t entry = 0;
#pragma unroll 1
        for (uint32_t step = 0; step < steps; ++step) {
            if (step < (uint32_t)order.count)
                entry = (uint32_t)(step < 5u ? order.packed[0] >> (12 * step) : order.packed[1] >> (12 * (step - 5u))) & 0xFFFu;
            else
                entry = step == (uint32_t)order.count || (entry & 15u) == INTERIOR ? kFirst : entry + kNext;
            group_solve<G, SUMS, Shape>(b, entry, lane);
        }
    } else {
        constexpr TeamGreedy greedy = team_greedy<S>();
        static_assert(greedy.steps <= 5, "12 bits per step");
        const bool second = (lane & (uint32_t)G) != 0u;
        const uint64_t packed_first = sweeps > 0u ? packed_entries(greedy, 0, true) : packed_entries(greedy, 0, false);
        constexpr uint64_t packed_second = packed_entries(greedy, 1, false);
        uint64_t ahead = second ? packed_second : packed_first;
#pragma unroll 1
        for (int step = 0; step < greedy.steps; ++step) {
            group_solve<G, SUMS, Shape>(b, (uint32_t)ahead & 0xFFFu, lane);
            ahead >>= 12;
        }
        uint32_t t = (uint32_t)greedy.head;  // (the first pair begins behind its head start)
#pragma unroll 1
        for (uint32_t left = sweeps; left > 0u;) {
            const bool pair = left > 1u;
            const uint32_t end = INTERIOR + (pair ? 2u : 0u), mine = second ? 2u : 0u;
#pragma unroll 1
            for (; t < end; ++t) {
                const uint32_t at = t - mine;  // level at + 1 of this chain's sweep
                const bool active = at < INTERIOR && (pair || !second);
                group_solve<G, SUMS, Shape>(b, active ? at * kNext + kFirst : 0u, lane);
            }
            t = 0;
            left -= pair ? 2u : 1u;
        }
    }
}

// The same by direct solves, by CHAINS groups of 16 lanes per bucket; general(entry) takes a step that they leave, and returns group_solve's
// result.  With one chain several groups may share a bucket: they all do the same.  A bucket without elements (behind the gradient's last
// one) is in no step's way.
//
// Sweeps behind the second find most levels where they are: such a step ends as soon as that shows, and a sweep that changes no level ends the
// solves, as the next one would find the same neighbours (20 sweeps, mixture, every step to its end -> this: five levels, 4096 buckets of 2048
// 60.6 -> 21.8 us, eight, 12290 of 4096 364 -> 260).  The first two sweeps do not look for it: looking costs a call with eight levels and two
// sweeps 3 %.
template <int CHAINS, int S, class Shape, class General>
__device__ __forceinline__ void group_solve_levels_direct(const GroupBucket& b, bool finite, uint32_t sweeps, uint32_t lane, General general)
{
    constexpr uint32_t INTERIOR = S - 2, RECORD = sizeof(GroupLevel);
    constexpr uint32_t kNext = 0x111u, kFirst = 0x201u;  // (as above)
    const DirectBucket direct = direct_bucket(b, finite, lane);
    const uint64_t some = __ballot(b.len > 0u);
    const uint32_t levels = (uint32_t)(uintptr_t)(LdsLevel*)b.level;
    uint32_t tries = 2;  // (values that many elements share would send every step both ways)
    bool changed = false;
    auto solve = [&](auto skip, uint32_t left, uint32_t right, uint32_t level, uint64_t active, uint32_t entry) __attribute__((always_inline)) {
        if (tries != 0u && group_solve_direct<Shape, decltype(skip)::value>(direct, left, right, level, active & some, lane, changed)) return;
        const bool moved = general(entry);
        if constexpr (decltype(skip)::value) changed = changed || moved;
        if (tries > 0u) --tries;
    };
    const uint32_t first_sweeps = umin32(sweeps, 2u);
    if constexpr (CHAINS == 1) {
        auto solve_entry = [&](auto skip, uint32_t entry) __attribute__((always_inline)) {
            solve(skip, levels + RECORD * ((entry >> 4) & 15u), levels + RECORD * (entry >> 8), levels + RECORD * (entry & 15u), ~0ull, entry);
        };
        constexpr GreedyOrder order = greedy_order<S>();
        static_assert(order.count <= 5, "12 bits per step");
        const uint32_t steps = (uint32_t)order.count + first_sweeps * INTERIOR;
        uint32_t entry = 0;
#pragma unroll 1
        for (uint32_t step = 0; step < steps; ++step) {
            if (step < (uint32_t)order.count) entry = (uint32_t)(order.packed[0] >> (12 * step)) & 0xFFFu;
            else entry = step == (uint32_t)order.count || (entry & 15u) == INTERIOR ? kFirst : entry + kNext;
            solve_entry(std::false_type{}, entry);
        }
#pragma unroll 1
        for (uint32_t left = sweeps - first_sweeps; left > 0u; --left) {
            changed = false;
#pragma unroll 1
            for (entry = kFirst; entry < kFirst + INTERIOR * kNext; entry += kNext) solve_entry(std::true_type{}, entry);
            if (!changed) break;
        }
    } else {
        constexpr uint64_t kChain[2] = {0x0000FFFF0000FFFFull, 0xFFFF0000FFFF0000ull};  // lanes
        const bool second = (lane & 16u) != 0u;
        constexpr TeamGreedy greedy = team_greedy<S>();
        static_assert(greedy.steps <= 5, "12 bits per step");
        constexpr uint64_t second_entries = packed_entries(greedy, 1, false);
        uint64_t first_ahead = sweeps > 0u ? packed_entries(greedy, 0, true) : packed_entries(greedy, 0, false), second_ahead = second_entries;
#pragma unroll 1
        for (int step = 0; step < greedy.steps; ++step) {
            const uint32_t e0 = (uint32_t)first_ahead & 0xFFFu, e1 = (uint32_t)second_ahead & 0xFFFu;
            const uint64_t active = (e0 != 0u ? kChain[0] : 0u) | (e1 != 0u ? kChain[1] : 0u);
            const uint32_t entry = second ? e1 : e0;
            solve(std::false_type{}, levels + RECORD * ((entry >> 4) & 15u), levels + RECORD * (entry >> 8),
                  levels + RECORD * (entry != 0u ? entry & 15u : (uint32_t)S), active, entry);
            first_ahead >>= 12;
            second_ahead >>= 12;
        }
        const uint32_t left_of_first = levels - (second ? 2u * RECORD : 0u);
        auto sweep = [&](auto skip, uint32_t t, bool pair) __attribute__((always_inline)) {  // one, or a pair
            const uint32_t end = INTERIOR + (pair ? 2u : 0u);
#pragma unroll 1
            for (; t < end; ++t) {
                const uint64_t active = (t < INTERIOR ? kChain[0] : 0u) | (pair && t >= 2u ? kChain[1] : 0u);
                const bool mine = __builtin_amdgcn_inverse_ballot_w64(active);
                const uint32_t at = left_of_first + RECORD * t;
                solve(skip, at, at + 2u * RECORD, mine ? at + RECORD : levels + RECORD * (uint32_t)S, active,
                      mine ? (second ? t - 2u : t) * kNext + kFirst : 0u);
            }
        };
        if (sweeps > 0u) sweep(std::false_type{}, (uint32_t)greedy.head, sweeps > 1u);  // (begins behind its head start)
#pragma unroll 1
        for (uint32_t left = sweeps - first_sweeps; left > 0u; left -= umin32(left, 2u)) {
            changed = false;
            sweep(std::true_type{}, 0u, left > 1u);
            if (!changed) break;
        }
    }
}

}  // namespace ogq
#endif  // OGQ_GROUP_SOLVE_H
