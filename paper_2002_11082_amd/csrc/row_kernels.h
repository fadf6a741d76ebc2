// Internal header of libogq: the random-rounding quantize kernels for small buckets of long gradients, four buckets per
// wavefront.  Included by rounding_part.hip after rounding_kernels.h, whose binning, exact sums and encoder it uses.
// Compile with -ffp-contract=off.
#ifndef OGQ_ROW_KERNELS_H
#define OGQ_ROW_KERNELS_H

#include "group_solve.h"

namespace ogq {

// ----------------------------------------------------------------------------------------------
// ORQ, Linear-s and evenly spaced levels for bucket sizes d = 64 m up to 512, four whole buckets per wavefront: row r (16
// lanes) owns bucket r of the wavefront's span of 4 d elements and holds its elements 64c + 4i + {0..3} in lane i, chunk c.
//
// What bounds it: vector-instruction issue (ORQ-9, buckets of 512, clipping, 25.6 M values: 3,337 vector instructions per
// wavefront at 2.2 ns per SIMD, SQ_ACTIVE_INST_VALU / SQ_BUSY_CU_CYCLES 0.96; ORQ-3, buckets of 128: 573 at 1.9 ns, 1.16).  With
// one bucket per wavefront (orq_quantize_kernel) a bucket of 512 elements costs 1,400 instructions at nine levels, of
// which its 8 x 64 elements need about 350: the solves, reductions and scans are the same for 2048 elements as for 512,
// and in a solve all 64 lanes do one bucket's arithmetic.  Here every such instruction works for four buckets: 834 per
// bucket.  25.6 M values, before -> after: ORQ-9 with clipping and the decoding of four workers 163 -> 105 us, ORQ-3 in
// buckets of 128 69 -> 44.  The phases are those of orq_bucket: extremes, grouping in LDS by value bins, fp64
// prefix, level solves, encode.  What differs: reductions and scans stay inside a row; bins are twice as wide (a bucket of
// 512 elements has at most about 20 elements in one), and the elements of the wanted bin are sorted across the row's 16
// lanes, one, two or four keys per lane.
//
// Positions and bin counts are kept in bytes (times 4), bin starts as LDS addresses, so that the scatter needs one
// addition per element.
// ----------------------------------------------------------------------------------------------
constexpr uint32_t kRows = 4, kRowLanes = 16;

// Per level: what OrqLds keeps; the sum of the elements not above the level follows from the others.
struct RowLevel {
    double sum_lt;
    float value;
    uint16_t count_lt, count_le;
    __device__ __forceinline__ double sum_le() const { return sum_lt + (double)(uint32_t)(count_le - count_lt) * (double)value; }
};

// LDS of a wavefront.  At 512 elements per bucket it decides how many wavefronts a CU holds (14 with 11 KB), so the bin
// counts give their place to the bin starts (half as wide) and the prefix once they are summed.
template <int C, int S>
struct RowLds {
    static constexpr int D = 64 * C;    // element capacity of a row
    static constexpr int B = 128;       // bins: 64 per sign, 4 per binade
    static constexpr int SHIFT = 21;    // magnitude bits dropped by the bin index
    static constexpr int BINS = B + 4;  // from row to row; entry B = end of the last bin
    static constexpr int BLOCK = D >= 512 ? 16 : 8;  // positions per entry of the fp64 prefix
    uint32_t grouped[kRows * D];        // fp32 bit patterns by bin, row after row
    union {
        uint32_t bin_count[kRows * BINS];  // bytes: 4 per element
        struct {
            double prefix[kRows * (D / BLOCK)];
            uint16_t bin_start[kRows * BINS];  // byte offset of each bin's first position in `grouped`
        };
    };
    RowLevel level[kRows][S];
    uint16_t level_rank[kRows][S];  // the rank a level was picked at (0 = not picked by rank)
    unsigned long long exact_limb[kRows][kExactLimbs];
};

__device__ __forceinline__ uint32_t row_inclusive_scan_u32(uint32_t x)
{
    x += dpp_or_zero_u32<kDppRowShr1, 0xF>(x);
    x += dpp_or_zero_u32<kDppRowShr2, 0xF>(x);
    x += dpp_or_zero_u32<kDppRowShr4, 0xF>(x);
    x += dpp_or_zero_u32<kDppRowShr8, 0xF>(x);
    return x;
}

// exact_floor_t of a row: its elements lie at grouped[0 .. len).
static __device__ __attribute__((noinline)) uint32_t exact_floor_t_row(unsigned long long* limb, const uint32_t* grouped,
                                                                       uint32_t len, uint32_t lane_in_row, float L, float R,
                                                                       uint32_t count_in, uint32_t guess)
{
    return exact_floor_t(limb, lane_in_row, kRowLanes, L, R, count_in, guess, [&](auto add) {
        for (uint32_t i = lane_in_row; i < len; i += kRowLanes) add(__uint_as_float(grouped[i]) + 0.0f);
    });
}

// Ascending sorts of K keys per lane over every row: element K * (lane in row) + register.
template <int J>
__device__ __forceinline__ void row_sort_across2(uint32_t (&x)[2], uint32_t lane)
{
    if constexpr (J >= 1) {
        const uint32_t bound = upper_lanes<J>(lane);
#pragma unroll
        for (int r = 0; r < 2; ++r) x[r] = smaller_or_larger(x[r], lane_xor<J>(x[r], lane), bound);
        row_sort_across2<J / 2>(x, lane);
    }
}

template <int M>
__device__ __forceinline__ void row_sort_merge2(uint32_t (&x)[2], uint32_t lane)
{
    if constexpr (2 * M <= (int)kRowLanes) {
        const uint32_t bound = upper_lanes<M>(lane);
        const uint32_t y0 = lane_reverse<M>(x[1], lane), y1 = lane_reverse<M>(x[0], lane);
        x[0] = smaller_or_larger(x[0], y0, bound);
        x[1] = smaller_or_larger(x[1], y1, bound);
        row_sort_across2<M / 2>(x, lane);
        sort_pair(x[0], x[1]);
        row_sort_merge2<2 * M>(x, lane);
    }
}

template <int K>
__device__ __forceinline__ void row_sort_keys(uint32_t (&x)[K], uint32_t lane)
{
    if constexpr (K == 1) {
        x[0] = wave_sort_merge<1>(x[0], lane);
        x[0] = wave_sort_merge<2>(x[0], lane);
        x[0] = wave_sort_merge<4>(x[0], lane);
        x[0] = wave_sort_merge<8>(x[0], lane);
    } else if constexpr (K == 2) {
        sort_pair(x[0], x[1]);
        row_sort_merge2<1>(x, lane);
    } else {
        row_sort<(int)kRowLanes>(x, lane);
    }
}

// An element picked by rank, the same in all lanes of a row (counts and sums are those of the row's bucket).
struct RowPicked {
    float value;
    uint32_t count_lt, count_le;
    double sum_lt;
};

// The element of index `index` (0-based) among the n (at most 16 K) values at byte offset `base` of the grouped array, which
// are the last elements in front of the wanted bin, if any, and the bin's own; counts and the sum are those within the n.
template <int K, bool SUMS, class Lds>
__device__ __forceinline__ RowPicked row_pick_sorted(const Lds& lds, uint32_t base, uint32_t n, uint32_t index, uint32_t lane)
{
    const uint32_t i = lane & (kRowLanes - 1u);
    const char* at = reinterpret_cast<const char*>(lds.grouped) + base + 4u * i;
    float value[K];
    uint32_t mine[K], x[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        // (a lane past the n reads whatever of the LDS record follows and drops it)
        value[k] = __uint_as_float(*reinterpret_cast<const uint32_t*>(at + 4u * kRowLanes * k)) + 0.0f;
        mine[k] = i + kRowLanes * k < n ? float_to_key(value[k]) : 0xFFFFFFFFu;
        x[k] = mine[k];
    }
    row_sort_keys<K>(x, lane);
    uint32_t source = x[0];
    if constexpr (K == 2) source = (index & 1u) ? x[1] : x[0];
    if constexpr (K == 4) {
        const uint32_t lo = (index & 1u) ? x[1] : x[0], hi = (index & 1u) ? x[3] : x[2];
        source = (index & 2u) ? hi : lo;
    }
    const uint32_t key = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(((lane & 48u) + index / (uint32_t)K) << 2), (int)source);
    RowPicked p{key_to_float(key), 0u, 0u, 0.0};
    if constexpr (SUMS) {
        uint32_t counts = 0;
        double part = 0.0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool below = mine[k] < key;
            counts += (below ? 1u : 0u) + (mine[k] <= key ? 0x10000u : 0u);
            part += (double)(below ? value[k] : 0.0f);
        }
        counts = row_sum_u32<(int)kRowLanes>(counts, lane);
        p.count_lt = counts & 0xFFFFu;
        p.count_le = umin32(counts >> 16, n);  // (a key of all ones, a NaN, equals the padding)
        p.sum_lt = row_sum_f64<(int)kRowLanes>(part, lane);
    }
    return p;
}

// The same for a crowded bin (some row's n is above 64): the key is found by bisection over the bits in which any row's
// smallest and largest key of the bin differ (none when all its values are equal).  rank: 1-based, inside the bin
// [first, last) (byte offsets); `front` elements lie in front of it.
template <bool SUMS, class Lds>
__device__ __forceinline__ RowPicked row_pick_bisected(const Lds& lds, uint32_t first, uint32_t last, uint32_t front, uint32_t rank,
                                                       uint32_t lane)
{
    const uint32_t i = lane & (kRowLanes - 1u);
    const char* grouped = reinterpret_cast<const char*>(lds.grouped);
    auto each = [&](uint32_t from, auto f) {
        for (uint32_t p = from + 4u * i; p < last; p += 4u * kRowLanes)
            f(__uint_as_float(*reinterpret_cast<const uint32_t*>(grouped + p)) + 0.0f);
    };
    uint32_t smallest = 0xFFFFFFFFu, largest = 0u;
    each(first, [&](float x) {
        smallest = umin32(smallest, float_to_key(x));
        largest = umax32(largest, float_to_key(x));
    });
    smallest = row_min_u32<(int)kRowLanes>(smallest, lane);
    largest = row_max_u32<(int)kRowLanes>(largest, lane);
    const uint32_t differing = smallest ^ largest;
    const uint32_t any = uniform_u32(wave_max_u32(differing));
    uint32_t key = smallest;
    if (any != 0u) {
        const int top = 31 - __builtin_clz(any);
        key = top == 31 ? 0u : smallest & ~((2u << top) - 1u);
#pragma unroll 1
        for (int bit = top; bit >= 0; --bit) {
            const uint32_t candidate = key | (1u << bit);
            uint32_t below = 0;
            each(first, [&](float x) { below += float_to_key(x) < candidate ? 1u : 0u; });
            below = row_sum_u32<(int)kRowLanes>(below, lane);
            if (below < rank) key = candidate;
        }
    }
    RowPicked p{key_to_float(key), 0u, 0u, 0.0};
    if constexpr (SUMS) {
        uint32_t counts = 0;
        double part = 0.0;
        each(first - 4u * front, [&](float x) {
            const bool below = float_to_key(x) < key;
            counts += (below ? 1u : 0u) + (float_to_key(x) <= key ? 0x10000u : 0u);
            part += (double)(below ? x : 0.0f);
        });
        counts = row_sum_u32<(int)kRowLanes>(counts, lane);
        p.count_lt = counts & 0xFFFFu;
        p.count_le = counts >> 16;
        p.sum_lt = row_sum_f64<(int)kRowLanes>(part, lane);
    }
    return p;
}

// The element of 1-based rank `rank` (1 .. bucket length) of every row's bucket.  coarse = start of the lane's first bin.
template <bool SUMS, class Lds>
__device__ __forceinline__ RowPicked row_pick(const Lds& lds, uint32_t rank, uint32_t coarse, uint32_t lane)
{
    constexpr uint32_t PER = Lds::B / kRowLanes;  // bins per lane: 8
    const uint32_t row = lane >> 4, i = lane & (kRowLanes - 1u);
    const uint32_t row_base = row * (4u * Lds::D);
    const uint32_t wanted = row_base + 4u * rank;  // the bin is the last one that starts below this
    const uint16_t* bins = lds.bin_start + row * Lds::BINS;
    const uint32_t segment = row_count(coarse < wanted, lane) - 1u;
    const uint32_t fine = bins[segment * PER + (i & (PER - 1u))];
    const uint32_t bin = segment * PER + row_count(i < PER && fine < wanted, lane) - 1u;
    const uint32_t first = bins[bin], last = bins[bin + 1u];

    const uint32_t position = (first - row_base) >> 2;
    const uint32_t front = SUMS ? position & (Lds::BLOCK - 1u) : 0u;
    double before = 0.0;
    if constexpr (SUMS) before = lds.prefix[row * (Lds::D / Lds::BLOCK) + position / Lds::BLOCK];
    const uint32_t n = front + ((last - first) >> 2), base = first - 4u * front;
    const uint32_t in_bin = rank - position;  // 1-based
    RowPicked p;
    if (__ballot(n > kRowLanes) == 0) p = row_pick_sorted<1, SUMS>(lds, base, n, front + in_bin - 1u, lane);
    else if (__ballot(n > 2u * kRowLanes) == 0) p = row_pick_sorted<2, SUMS>(lds, base, n, front + in_bin - 1u, lane);
    else if (__ballot(n > 4u * kRowLanes) == 0) p = row_pick_sorted<4, SUMS>(lds, base, n, front + in_bin - 1u, lane);
    else p = row_pick_bisected<SUMS>(lds, first, last, front, in_bin, lane);
    if constexpr (SUMS) {
        p.count_lt += position - front;
        p.count_le += position - front;
        p.sum_lt += before;
    }
    return p;
}

// One level solve of every row's bucket: level k between the levels l and r (see orq_solve_one).
template <bool SUMS, class Lds>
__device__ __forceinline__ void row_solve(Lds& lds, uint32_t k, uint32_t l, uint32_t r, uint32_t len, double bound, uint32_t coarse,
                                          uint32_t lane)
{
    const uint32_t row = lane >> 4, i = lane & (kRowLanes - 1u);
    const RowLevel left = lds.level[row][l], right = lds.level[row][r];
    const uint32_t last_rank = lds.level_rank[row][k];
    const float L = left.value, R = right.value;
    const bool ordered = L < R;
    // S = sum_{L<=v<=R} (v - L),  T = S / (R - L),  level = element of rank #{v<=R} - floor(T)
    const uint32_t count_in = right.count_le - left.count_lt;
    const double Ssum = (right.sum_le() - left.sum_lt) - (double)L * (double)count_in;
    const double width = (double)R - (double)L;
    double m;  // not used when L == R
    const bool decided = floor_t_from_sums(Ssum, width, bound, m);
    if (ordered && !decided)
        m = (double)exact_floor_t_row(lds.exact_limb[row], lds.grouped + row * Lds::D, len, i, L, R, count_in, (uint32_t)m);
    const uint32_t below = (uint32_t)fmin(m, 65536.0);
    uint32_t rank = below >= right.count_le ? 1u : right.count_le - below;
    rank = umin32(rank, len);
    const bool same = ordered && rank == last_rank;  // same element as last time
    if (__ballot(!same) == 0) return;
    const RowPicked p = row_pick<SUMS>(lds, rank, coarse, lane);
    const bool copy_left = !ordered || p.value < L;  // the level coincides with the left end
    RowLevel now;
    now.value = copy_left ? L : p.value;
    now.count_lt = (uint16_t)(copy_left ? left.count_lt : p.count_lt);
    now.count_le = (uint16_t)(copy_left ? (ordered ? left.count_le : right.count_le) : p.count_le);
    now.sum_lt = copy_left ? left.sum_lt : p.sum_lt;
    if (i == 0u && !same) {
        lds.level[row][k] = now;
        lds.level_rank[row][k] = (uint16_t)(copy_left ? 0u : rank);
    }
    wave_lds_sync();
}

// The reload function of the encoder: g = the row's first element, limit = its clipping threshold (infinity: none).
struct ReloadRow {
    const float* g;
    float limit;
    __device__ __forceinline__ void operator()(uint32_t c, float (&y)[4]) const
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = fminf(fmaxf(g[64u * c + 4u * (threadIdx.x & 15u) + (uint32_t)k], -limit), limit);
    }
};

// Runs f(c) for the chunks of a row: c < chunks, all C of them where EXACT.
template <int C, bool EXACT, class F>
__device__ __forceinline__ void for_row_chunks(uint32_t chunks, F f)
{
#pragma unroll
    for (int c = 0; c < C; ++c)
        if (EXACT || (uint32_t)c < chunks) f(c);
}

// The four whole buckets of `chunks` * 64 elements that begin at global element `begin`; bucket = the first one's index.
template <int C, int S, int BITS, bool EXACT, int RULE>
__device__ __forceinline__ void orq_rows_span(RowLds<C, S>& lds, const float* __restrict__ grad, uint32_t chunks, size_t begin,
                                              uint32_t bucket, uint32_t sweeps, float clip, uint64_t seed, uint64_t index_offset,
                                              float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    static_assert(RULE == kOptimal || RULE == kEven || RULE == kLinear, "rules of this kernel");
    using Lds = RowLds<C, S>;
    constexpr uint32_t B = Lds::B, HALF = B / 2;
    constexpr uint32_t PER = B / kRowLanes;
    constexpr bool GROUPED = S > 2 && RULE != kEven;
    constexpr bool SUMS = RULE == kOptimal && S > 3;  // with one interior level the solve reads the bucket's total alone
    const uint32_t lane = threadIdx.x & 63u, row = lane >> 4, i = lane & (kRowLanes - 1u);
    const uint32_t len = 64u * chunks;
    const float* g = grad + begin + row * len;

    float v[C][4];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[c][k] = 0.0f;
    for_row_chunks<C, EXACT>(chunks, [&](int c) {
        const floatx4 q = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(g + 64 * c + 4 * i));
        v[c][0] = q.x; v[c][1] = q.y; v[c][2] = q.z; v[c][3] = q.w;
    });
    float limit = __uint_as_float(0x7F800000u);  // clipping threshold
    if (clip > 0.0f) {  // the same for every thread of the grid
        float(&flat)[4 * C] = reinterpret_cast<float(&)[4 * C]>(v);
        limit = clip_in_registers<4 * C>(
            flat, len, clip, [&](int j) { return EXACT || (uint32_t)(j >> 2) < chunks; },
            [&](double x) { return row_sum_f64<(int)kRowLanes>(x, lane); });
    }

    // ---- extremes of every row ---------------------------------------------------------------------
    float low = v[0][0], high = v[0][0];
    for_row_chunks<C, EXACT>(chunks, [&](int c) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            low = fminf(low, v[c][k]);
            high = fmaxf(high, v[c][k]);
        }
    });
    low = key_to_float(row_min_u32<(int)kRowLanes>(float_to_key(low + 0.0f), lane));  // (-0 -> +0)
    high = key_to_float(row_max_u32<(int)kRowLanes>(float_to_key(high + 0.0f), lane));
    const uint32_t mag_max = umax32(__float_as_uint(low) & 0x7FFFFFFFu, __float_as_uint(high) & 0x7FFFFFFFu);

    if constexpr (GROUPED) {
        const uint32_t t_low = __builtin_elementwise_sub_sat(mag_max >> Lds::SHIFT, HALF - 1u);
        const uint32_t row_bins = row * (4u * Lds::BINS);  // bytes
        const uint32_t row_base = row * (4u * Lds::D);
        char* bins = reinterpret_cast<char*>(lds.bin_count);
        uint4* my_bins = reinterpret_cast<uint4*>(bins + row_bins + 4u * PER * i);
        my_bins[0] = make_uint4(0u, 0u, 0u, 0u);
        my_bins[1] = make_uint4(0u, 0u, 0u, 0u);
        wave_lds_sync();

        // ---- histogram: the returning LDS add hands every element its position inside its bin --------
        uint32_t slot[C][4];  // byte offset of the bin's counter | 4 * position inside the bin << 16
        const float zero = opaque_zero();
        for_row_chunks<C, EXACT>(chunks, [&](int c) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t at = value_bin<(int)HALF, Lds::SHIFT>(v[c][k] + zero, t_low) * 4u + row_bins;
                slot[c][k] = __builtin_amdgcn_perm(atomicAdd(reinterpret_cast<uint32_t*>(bins + at), 4u), at, 0x05040100u);
            }
        });
        wave_lds_sync();

        // ---- bin starts: exclusive prefix over the row's counts (lane i owns PER bins) ----------------
        uint32_t coarse;
        {
            const uint4 a = my_bins[0], b = my_bins[1];
            wave_lds_sync();  // all counts are read before the starts take their place
            const uint32_t total = (a.x + a.y) + (a.z + a.w) + (b.x + b.y) + (b.z + b.w);
            coarse = row_base + row_inclusive_scan_u32(total) - total;
            uint32_t start[PER + 1] = {coarse};
            const uint32_t count[PER] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (uint32_t t = 0; t < PER; ++t) start[t + 1] = start[t] + count[t];
            uint32_t* pairs = reinterpret_cast<uint32_t*>(lds.bin_start + row * Lds::BINS) + PER / 2u * i;
#pragma unroll
            for (uint32_t t = 0; t < PER / 2u; ++t) pairs[t] = start[2u * t] | start[2u * t + 1u] << 16;
            if (i == kRowLanes - 1u) lds.bin_start[row * Lds::BINS + B] = (uint16_t)start[PER];  // = row_base + 4 len
        }
        wave_lds_sync();

        // ---- scatter the values into their bins (bin starts of a group of chunks read before its writes) ----
        char* grouped = reinterpret_cast<char*>(lds.grouped);
        const char* starts = reinterpret_cast<const char*>(lds.bin_start);
        constexpr int GROUP = C < 4 ? C : 4;
#pragma unroll
        for (int c0 = 0; c0 < C; c0 += GROUP) {
#pragma unroll
            for (int c = c0; c < c0 + GROUP; ++c)
                if (EXACT || (uint32_t)c < chunks) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        slot[c][k] = *reinterpret_cast<const uint16_t*>(starts + __builtin_amdgcn_ubfe(slot[c][k], 1u, 15u)) +
                                     (slot[c][k] >> 16);  // (a start is half as wide as a counter)
                }
#pragma unroll
            for (int c = c0; c < c0 + GROUP; ++c)
                if (EXACT || (uint32_t)c < chunks) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        *reinterpret_cast<uint32_t*>(grouped + slot[c][k]) = __float_as_uint(v[c][k]);
                }
        }
        wave_lds_sync();

        // ---- fp64 prefix of the grouped values, one entry per BLOCK positions (lane i: 4 C positions) ------
        double total = 0.0, bound = 0.0;
        if constexpr (SUMS) {
            constexpr uint32_t MINE = 4u * C, BLOCK = Lds::BLOCK;
            const float4* from = reinterpret_cast<const float4*>(lds.grouped + row * Lds::D + MINE * i);
            double part = 0.0, before[MINE / BLOCK > 0 ? MINE / BLOCK : 1];
#pragma unroll
            for (uint32_t q = 0; q < (uint32_t)C; ++q) {
                if (4u * q % BLOCK == 0u) before[4u * q / BLOCK] = part;
                const bool exists = EXACT || MINE * i + 4u * q < len;
                const float4 x = from[q];
                part += (double)(exists ? x.x : 0.0f);
                part += (double)(exists ? x.y : 0.0f);
                part += (double)(exists ? x.z : 0.0f);
                part += (double)(exists ? x.w : 0.0f);
            }
            const double incl = row_inclusive_scan_f64<(int)kRowLanes>(part);
            double* entry = lds.prefix + row * (Lds::D / BLOCK) + MINE / BLOCK * i;
            if constexpr (MINE >= BLOCK) {
#pragma unroll
                for (uint32_t q = 0; q < MINE / BLOCK; ++q) entry[q] = (incl - part) + before[q];
            } else {
                // (C = 1: two lanes share an entry)
                if (i % (BLOCK / MINE) == 0u) lds.prefix[row * (Lds::D / BLOCK) + i / (BLOCK / MINE)] = incl - part;
            }
            total = lane_fetch_f64(incl, lane | (kRowLanes - 1u));
        } else if constexpr (RULE == kOptimal) {
            double part = 0.0;
            for_row_chunks<C, EXACT>(chunks, [&](int c) {
#pragma unroll
                for (int k = 0; k < 4; ++k) part += (double)v[c][k];
            });
            total = row_sum_f64<(int)kRowLanes>(part, lane);
        }

        if constexpr (RULE == kOptimal) {
            // ---- may the fp64 sums round?  (small elements sit in the bins next to zero: see any_tiny_element) ----
            constexpr uint32_t SAFE = safe_binades(Lds::D);
            const uint32_t biased = mag_max >> 23;
            bool tiny = false;
            if (biased > SAFE) {
                const uint32_t mag_safe = (biased - SAFE) << 23;
                const uint32_t t_safe = mag_safe >> Lds::SHIFT;
                const uint32_t near = umin32(t_safe > t_low ? t_safe - t_low : 1u, HALF);
                const uint16_t* row_bin = lds.bin_start + row * Lds::BINS;
                const uint32_t last = row_bin[HALF + near];
                for (uint32_t p = row_bin[HALF - near] + 4u * i; p < last; p += 4u * kRowLanes) {
                    const uint32_t magnitude = *reinterpret_cast<const uint32_t*>(grouped + p) & 0x7FFFFFFFu;
                    tiny = tiny || (magnitude != 0u && magnitude < mag_safe);
                }
            }
            bound = row_count(tiny, lane) != 0u ? sum_error_bound_of(mag_max, Lds::D) : 0.0;
        }
        // ---- level records of the ends -------------------------------------------------------------------
        if (i < (uint32_t)S) {
            const bool top = i == (uint32_t)(S - 1);
            RowLevel end;
            end.value = top ? high : low;
            end.count_lt = end.count_le = (uint16_t)(top ? len : 0u);
            end.sum_lt = top ? total : 0.0;
            lds.level[row][i] = end;
            lds.level_rank[row][i] = 0u;
        }
        wave_lds_sync();

        // ---- the levels ------------------------------------------------------------------------------------
        if constexpr (RULE == kLinear) {
#pragma unroll 1
            for (uint32_t k = 1; k + 1 < (uint32_t)S; ++k) {
                const RowPicked p = row_pick<false>(lds, 1u + k * (len - 1u) / (uint32_t)(S - 1), coarse, lane);
                if (i == 0u) lds.level[row][k].value = p.value;
            }
            wave_lds_sync();
        } else {
            constexpr GreedyOrder order = greedy_order<S>();
            const uint32_t steps = order.count + (S > 3 ? sweeps * (S - 2) : 0u);  // (one interior level: sweeps repeat it)
#pragma unroll 1
            for (uint32_t step = 0; step < steps; ++step) {
                uint32_t k, l, r;
                if (step < (uint32_t)order.count) {
                    const uint32_t e = step < 5u ? (uint32_t)(order.packed[0] >> (12 * step))
                                                 : (uint32_t)(order.packed[1] >> (12 * (step - 5u)));
                    k = e & 15u; l = (e >> 4) & 15u; r = (e >> 8) & 15u;
                } else {
                    k = 1u + (step - order.count) % (S - 2);
                    l = k - 1u; r = k + 1u;
                }
                row_solve<SUMS>(lds, k, l, r, len, bound, coarse, lane);
            }
        }
    }

    float lv[S];
    if constexpr (RULE == kEven) {
        const double largest = (double)__uint_as_float(mag_max);
#pragma unroll
        for (int k = 0; k < S; ++k) lv[k] = (float)(largest * (double)(2 * k - (S - 1)) / (double)(S - 1));
    } else {
        lv[0] = low;
        lv[S - 1] = high;
#pragma unroll
        for (int k = 1; k < S - 1; ++k) lv[k] = lds.level[row][k].value;
    }
    float mine = lv[0];
#pragma unroll
    for (int k = 1; k < S; ++k) mine = i == (uint32_t)k ? lv[k] : mine;
    if (i < (uint32_t)S) levels[(size_t)(bucket + row) * S + i] = mine;

    const EncodeRange range{256u * chunks, (index_offset + begin) >> 2, row * (len / 4u) + i, chunks, (uint32_t)seed,
                            (uint32_t)(seed >> 32), codes32 + begin / 64 * (2 * BITS)};
    encode_all<FourRows, C, S, BITS, EXACT ? Fill::kAll : Fill::kWholeChunks>(v, lv, range, ReloadRow{g, limit});
}

// Blocks 0 .. singles - 1 take the buckets behind the last whole span (at most three whole ones and a cut-off one), one
// each as in orq_quantize_kernel and first so that they do not end the launch alone; the others take a span each.
template <int C, int S, int BITS, bool EXACT, int RULE>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(C == 8 ? (EXACT ? 4 : 3) : 1))) void orq_rows_kernel(const float* __restrict__ grad, size_t n, uint32_t bucket_size,
                                                         uint32_t sweeps, float clip, uint32_t num_buckets, uint32_t spans,
                                                         uint64_t seed, uint64_t index_offset, float* __restrict__ levels,
                                                         uint32_t* __restrict__ codes32)
{
    constexpr int CB = C <= 4 ? 1 : 2;  // chunks of 256 elements of a bucket
    using Single = OrqLds<OrqShape<CB>::D, OrqShape<CB>::B, S>;
    using Rows = RowLds<C, S>;
    __shared__ __attribute__((aligned(16))) unsigned char raw[sizeof(Rows) > sizeof(Single) ? sizeof(Rows) : sizeof(Single)];
    const uint32_t singles = num_buckets - kRows * spans;
    if (blockIdx.x < singles) {
        const uint32_t bucket = kRows * spans + blockIdx.x;
        const size_t begin = (size_t)bucket * bucket_size;
        const size_t rest = n - begin;
        const uint32_t len = rest < bucket_size ? (uint32_t)rest : bucket_size;
        orq_bucket<CB, S, BITS, false, true, RULE>(*reinterpret_cast<Single*>(raw), grad + begin, len, begin, bucket, sweeps, clip,
                                                   seed, index_offset, levels, codes32);
    } else {
        const uint32_t bucket = kRows * (blockIdx.x - singles);
        orq_rows_span<C, S, BITS, EXACT, RULE>(*reinterpret_cast<Rows*>(raw), grad, bucket_size / 64u, (size_t)bucket * bucket_size,
                                               bucket, sweeps, clip, seed, index_offset, levels, codes32);
    }
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------
template <int C, int S, int BITS, bool EXACT, int RULE>
void launch_rows(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    const uint32_t spans = (uint32_t)(n / p->bucket_size / kRows);
    launch_kernel((orq_rows_kernel<C, S, BITS, EXACT, RULE>), dim3(nb - kRows * spans + spans), dim3(kWave), st, g, n, p->bucket_size,
                  p->level_iters, p->clip_factor, nb, spans, p->seed, p->index_offset, lv, static_cast<uint32_t*>(codes));
}

template <int C, bool EXACT>
bool launch_rows_levels(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    switch (p->scheme) {
        case OGQ_ORQ:
            switch (p->bits) {
                case 1: launch_rows<C, 2, 1, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
                case 2: launch_rows<C, 4, 2, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
                default: launch_rows<C, 8, 3, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
            }
        case OGQ_ORQ_PAPER:
            switch (p->bits) {
                case 2: launch_rows<C, 3, 2, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
                case 3: launch_rows<C, 5, 3, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
                default: launch_rows<C, 9, 4, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
            }
        case OGQ_EVEN:
            switch (p->bits) {
                case 2: launch_rows<C, 3, 2, EXACT, kEven>(g, n, p, nb, lv, codes, st); return true;
                case 3: launch_rows<C, 5, 3, EXACT, kEven>(g, n, p, nb, lv, codes, st); return true;
                default: launch_rows<C, 9, 4, EXACT, kEven>(g, n, p, nb, lv, codes, st); return true;
            }
        case OGQ_LINEAR:
            switch (p->bits) {
                case 2: launch_rows<C, 3, 2, EXACT, kLinear>(g, n, p, nb, lv, codes, st); return true;
                case 3: launch_rows<C, 5, 3, EXACT, kLinear>(g, n, p, nb, lv, codes, st); return true;
                default: launch_rows<C, 9, 4, EXACT, kLinear>(g, n, p, nb, lv, codes, st); return true;
            }
        default: return false;  // BinGrad-pb
    }
}

}  // namespace ogq
#endif  // OGQ_ROW_KERNELS_H
