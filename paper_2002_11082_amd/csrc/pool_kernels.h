// Internal header of libogq: the random-rounding quantize kernel for buckets of 513 to 4096 elements whose rule solves several
// interior levels (ORQ with four levels and more), two or four buckets per workgroup.  Included by rounding_part.hip after
// rounding_kernels.h, whose exact sums and encoder it uses.  Compile with -ffp-contract=off.
#ifndef OGQ_POOL_KERNELS_H
#define OGQ_POOL_KERNELS_H

#include "group_solve.h"

namespace ogq {

// ----------------------------------------------------------------------------------------------
// Two or four buckets per workgroup, W wavefronts each, wavefront w of a bucket holding its elements [256 C w, 256 C (w + 1)) in the
// register layout of orq_bucket.  The phases are those of orq_team_kernel: load, extremes, grouping in LDS, fp64 prefix, level solves,
// encode; but one wavefront of the workgroup solves the levels of all side by side, a row of 16 lanes for each of a
// bucket's two chains of solves (group_solve.h), which begin with Algorithm 1's second level; four levels are one chain.
//
// A solve is some 120 vector instructions on values that are the same for the whole bucket, in one chain of LDS reads and
// fp64 operations.  With a wavefront's 64 lanes on one solve (orq_team_kernel), eight levels and two sweeps took 11 steps behind workgroup
// barriers and most of a wavefront's scalar instructions; here the four rows work for two buckets and the steps need no barrier.
// 143.7 M values in buckets of 4096, eight levels, two sweeps: 421 -> 368 us, with direct solves (group_solve_direct) and 1280 instead of 1024
// bins, so that hardly a bin is too large for them, 310; 25.6 M values in buckets of 2048 124 -> 80 -> 69.
// Bound by the solves' latency (profiles/phase_cycles.txt), of which the random numbers that a workgroup's other wavefronts make meanwhile are the
// smaller part, and the LDS (16 KB of values per bucket of 4096), which holds the buckets of four workgroups; the vector units are busy 0.88 of the time
// (profiles/orq_cfg4_issue_counters_pmc.txt).  The solving wavefront runs at a raised priority: its instructions go first on its SIMD.  Four
// buckets per workgroup, in rows of 8 lanes, were slower (418 us when two took 368): fewer workgroups overlap.
// Four levels: four buckets of up to 2048 elements, a row each, so that a workgroup spends no more instructions on solves than with more
// levels (25.6 M values in buckets of 2048, two sweeps, mean of four kinds of values: one wavefront per bucket 54.4 us, two buckets in a
// workgroup 50.9, four 50.7; 8192 buckets 38 / 37 / 32).  Above 2048 elements the LDS of a workgroup (an address in 16 bits) holds two, whose
// two rows do the same work.
// ----------------------------------------------------------------------------------------------
// Priorities of a wavefront.  The random numbers that a waiting wavefront makes are work for what the others leave: at the priority of all but the
// solves they held up the histograms and scatters of the CU's workgroups whose loads had come late, which end the call (1920 buckets of
// 4096, eight levels, two sweeps: bin starts 2,800 cycles in the slowest tenth of the workgroups, where they had taken 1,200).  us, no numbers ahead -> ahead, at
// work's priority -> below it: four levels, two sweeps, 1920 buckets of 2112 18.2 -> 19.0 -> 16.8, 1628 of 3072 19.1 -> 19.7 -> 17.5; eight levels, 1920 of
// 4096 23.5 -> 22.8 -> 21.6, 143.7 M values in buckets of 4096 313 -> 286 -> 273.
constexpr int kAhead = 0, kAtWork = 1, kSolving = 3;

constexpr int pool_chains(int S) { return S > 4 ? 2 : 1; }                     // of solves per bucket, a row of 16 lanes each
constexpr int pool_buckets(int W, int S) { return W == 1 && S == 4 ? 4 : 2; }  // per workgroup

template <int W, int C, int S>
struct alignas(16) PoolBucket {
    static constexpr int D = 256 * C * W;                      // element capacity
    static constexpr int B = C == 8 ? (W == 2 ? 5 * D / 16 : D / 4) : D / 2, HALF = B / 2;  // bins: what the LDS leaves room for
    static constexpr int BLOCK = 4 * C;                        // positions per entry of the fp64 prefix: one lane's
    static constexpr bool END_OF_BUCKET = false, LEAF = true;  // (group_solve)
    union {
        uint32_t bin_count[B];  // bytes: 4 per element
        uint32_t grouped[D];    // fp32 bit patterns by bin
    };
    double prefix[D / BLOCK];
    GroupLevel level[S + 1];    // (the last one takes what is of no use)
    double wave_sum[W];
    TeamSlot slots[2][W];
    uint16_t bin_start[B + 2];  // byte offset of each bin's first position in `grouped`; [B] = end of the last bin
    ScaledBins bins;
    uint32_t tiny;              // set where an element is too small for exact sums

    // What group_solve needs of a bucket of `len` elements.
    __device__ __forceinline__ GroupBucket view(unsigned long long* limb, uint32_t len)
    {
        const uint32_t largest = umax32(__float_as_uint(level[0].value) & 0x7FFFFFFFu, __float_as_uint(level[S - 1].value) & 0x7FFFFFFFu);
        return GroupBucket{reinterpret_cast<const char*>(grouped), bin_start + HALF, prefix, level, limb, bins, 0u, len,
                           tiny != 0u ? sum_error_bound_of(largest, (uint32_t)D) : 0.0};
    }
};

template <int W, int C, int S>
struct PoolLds {
    PoolBucket<W, C, S> bucket[pool_buckets(W, S)];
    unsigned long long exact_limb[kExactLimbs];
};

// A step of solves that group_solve_direct leaves (bucket, limb: LDS addresses).  Out of line: few steps take it.
template <class Bucket>
static __device__ __attribute__((noinline)) uint32_t pool_solve_general(uint32_t bucket, uint32_t limb, uint32_t len, uint32_t entry, uint32_t lane)
{
    Bucket& b = *(Bucket*)(__attribute__((address_space(3))) Bucket*)(uintptr_t)bucket;
    return group_solve<16, true, Bucket>(b.view((unsigned long long*)(__attribute__((address_space(3))) unsigned long long*)(uintptr_t)limb, len), entry, lane);
}

template <int W, int C, int S, int BITS, bool FULL>
__device__ __forceinline__ void orq_pool_group(PoolLds<W, C, S>& lds, const float* __restrict__ grad, size_t n,
                                               uint32_t bucket_size, uint32_t sweeps, float clip, uint32_t num_buckets, uint64_t seed,
                                               uint64_t index_offset, float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    static_assert(W == 1 || W == 2, "the bin starts of a second wavefront follow from its own total");
    using Bucket = PoolBucket<W, C, S>;
    constexpr uint32_t PER_WAVE = 256u * C, B = Bucket::B, HALF = Bucket::HALF, BLOCK = Bucket::BLOCK;
    constexpr int NB = pool_buckets(W, S);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = uniform_u32(threadIdx.x >> 6);
    const uint32_t slot_of = wave / (uint32_t)W, part = wave % (uint32_t)W;  // bucket of the workgroup, wavefront of the bucket
    const uint32_t bucket = blockIdx.x * (uint32_t)NB + slot_of;
    Bucket& my = lds.bucket[slot_of];
    const bool exists = FULL || bucket < num_buckets;
    const size_t begin = exists ? (size_t)bucket * bucket_size : 0u;
    uint32_t len = (uint32_t)Bucket::D;
    if constexpr (!FULL) {
        const size_t rest = n - begin;
        len = !exists ? 0u : rest < bucket_size ? (uint32_t)rest : bucket_size;
    }
    const float* g = grad + begin;
    const uint32_t first = PER_WAVE * part;
    const uint32_t my_len = FULL ? PER_WAVE : len > first ? (len - first < PER_WAVE ? len - first : PER_WAVE) : 0u;
    auto sync = [&]() __attribute__((always_inline)) {  // of the wavefronts that hold a bucket
        if constexpr (W == 1) wave_lds_sync();
        else __syncthreads();
    };

    __builtin_amdgcn_s_setprio(kAtWork);
    float v[C][4];
    load_range<C, FULL>(v, g, first, len, my_len, lane);
    uint32_t grouped_at = (uint32_t)(uintptr_t)((LdsWord*)my.grouped);
    asm("" : "+s"(grouped_at));
    {
        constexpr uint32_t ZEROS = B / (64u * W) / 2u;
        uint2* mine = reinterpret_cast<uint2*>(my.bin_count) + ZEROS * (64u * part + lane);
        const uint32_t count = counter_start((uint32_t)(uintptr_t)((LdsHalf*)my.bin_start), grouped_at, 2u * ZEROS * (64u * part + lane));
#pragma unroll
        for (uint32_t i = 0; i < ZEROS; ++i) mine[i] = make_uint2(count + (i << 18), count + (i << 18) + (1u << 17));
        if (part == 0u && lane == 0u) my.tiny = 0u;
    }
    WaveTeam<W> team{my.slots, part, 0u};

    float limit = __uint_as_float(0x7F800000u);  // clipping threshold
    if (clip > 0.0f) {  // the same for every thread of the grid
        float(&flat)[4 * C] = reinterpret_cast<float(&)[4 * C]>(v);
        uint32_t here = lane;
        limit = clip_in_registers<4 * C, (W > 1)>(
            flat, len, clip, [&](int j) { return FULL || (64u * (j & ~3) + 4u * here + (j & 3) < my_len); },
            [&](double& x, double& y) __attribute__((always_inline)) {
                if constexpr (!FULL) asm volatile("" : "+v"(here));  // (see set_padding)
                x = wave_sum(x);
                y = wave_sum(y);
                if constexpr (W > 1) team.sums(x, y);
            });
        if constexpr (!FULL) set_padding<C>(v, my_len, lane);
    }

    // ---- extremes of the bucket ------------------------------------------------------------------------
    float low, high;
    uint32_t unused_zeros;
    lane_extremes<C, false>(v, low, high, unused_zeros);
    wave_extremes(low, high);
    // mean magnitude of every fourth element (padding is NaN)
    float sample = 0.0f;
#pragma unroll
    for (int c = 0; c < C; ++c) sample += FULL || v[c][0] == v[c][0] ? __builtin_fabsf(v[c][0]) : 0.0f;
    double magnitudes = (double)wave_sum_f32(sample);
    if constexpr (W > 1) {
        const TeamSlot* s = team.exchange(magnitudes, __float_as_uint(low), __float_as_uint(high));
#pragma unroll
        for (int w = 0; w < W; ++w) {
            low = fminf(low, __uint_as_float(s[w].a));
            high = fmaxf(high, __uint_as_float(s[w].b));
        }
        magnitudes = s[0].sum + s[W - 1].sum;
    } else {
        wave_lds_sync();  // the zeroed bins
    }
    low = uniform_f32(low + 0.0f);  // -0 -> +0
    high = uniform_f32(high + 0.0f);
    const uint32_t mag_max = umax32(__float_as_uint(low) & 0x7FFFFFFFu, __float_as_uint(high) & 0x7FFFFFFFu);
    const float mean = (float)magnitudes * __builtin_amdgcn_rcpf((float)((len + 3u) / 4u));
    ScaledBins bins_of = scaled_bins<(int)HALF>(mean, mag_max);
    bins_of.factor = uniform_u32(bins_of.factor);

    // ---- histogram: the returning LDS add hands every element its position inside its bin ------------------
    uint32_t slot[C][4];  // what the bin's counter returned (counter_start)
    {
        const float zero = opaque_zero();
        const uint64_t origin = bin_origin(bins_of);
        uint32_t middle = (uint32_t)(uintptr_t)((LdsWord*)my.bin_count + HALF);
        asm("" : "+s"(middle));  // (one addition with the bin, not two)
        uint32_t here = lane;
        if constexpr (!FULL) asm volatile("" : "+v"(here));  // (see set_padding)
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (FULL || 256u * (uint32_t)c < my_len) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const bool valid = FULL || 256u * c + 4u * here + k < my_len;
                    // (padding adds 0 to one bin per lane: no branch)
                    const uint32_t counter = middle + 4u * (uint32_t)(valid ? signed_bin<(int)HALF>(v[c][k] + zero, bins_of, origin) : (int32_t)here);
                    slot[c][k] = __hip_atomic_fetch_add((LdsWord*)(uintptr_t)counter, valid ? 4u : 0u, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) slot[c][k] = 0u;
            }
        }
    }
    sync();

    // ---- bin starts: wavefront `part` owns the bins [part B / W, (part + 1) B / W) ---------------------------
    {
        constexpr uint32_t PER = B / (64u * W);  // bins per lane
        static_assert(PER % 2u == 0u, "8-byte reads");
        const uint2* mine = reinterpret_cast<const uint2*>(my.bin_count) + PER / 2u * (64u * part + lane);
        uint32_t count[PER], total = 0;
#pragma unroll
        for (uint32_t q = 0; q < PER / 2u; ++q) {
            const uint2 x = mine[q];
            count[2 * q] = x.x; count[2 * q + 1] = x.y;
        }
#pragma unroll
        for (uint32_t t = 0; t < PER; ++t) total += count[t];
        total -= PER * grouped_at;  // (the lower 16 bits are what counts)
        const uint32_t incl = wave_inclusive_scan_u32(total);
        uint32_t start = incl - total;
        if constexpr (W == 2)  // all counts together make the bucket
            start += part == 0u ? 0u : 4u * len - __builtin_amdgcn_readlane(incl, 63);
        uint32_t* pairs = reinterpret_cast<uint32_t*>(my.bin_start) + PER / 2u * (64u * part + lane);
#pragma unroll
        for (uint32_t t = 0; t < PER / 2u; ++t) {
            const uint32_t next = start + count[2 * t] - grouped_at;
            pairs[t] = two_starts(start, next);
            start = next + count[2 * t + 1] - grouped_at;
        }
        if (part == (uint32_t)W - 1u && lane == 63u) my.bin_start[B] = (uint16_t)start;  // = 4 len
    }
    sync();

    // ---- scatter the values into their bins (bin starts of a group of chunks read before its writes) ----------
    {
        constexpr int GROUP = 4;
        uint32_t here = lane;
        if constexpr (!FULL) asm volatile("" : "+v"(here));  // (see set_padding)
#pragma unroll
        for (int c0 = 0; c0 < C; c0 += GROUP) {
            if (!FULL && 256u * (uint32_t)c0 >= my_len) continue;
#pragma unroll
            for (int c = c0; c < c0 + GROUP; ++c)
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    slot[c][k] = place_in_bin(slot[c][k]);
#pragma unroll
            for (int c = c0; c < c0 + GROUP; ++c)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    uint32_t at = slot[c][k], bits = __float_as_uint(v[c][k]);
                    if constexpr (!FULL) {
                        // padding goes where it lies in the bucket, behind all elements, as zeros that the prefix may add
                        const uint32_t e = 256u * c + 4u * here + k;
                        const bool valid = e < my_len;
                        at = valid ? at : grouped_at + 4u * (first + e);
                        bits = valid ? bits : 0u;
                    }
                    *(LdsWord*)(uintptr_t)at = bits;
                }
        }
    }
    sync();

    // ---- fp64 prefix of the grouped values: a lane sums the BLOCK positions of one entry -----------------------
    {
        const float4* from = reinterpret_cast<const float4*>(my.grouped + PER_WAVE * part + BLOCK * lane);
        // every lane begins at another of its 16-byte pieces, so that the lanes meet different LDS banks
        const uint32_t turn = lane / (C < 8 ? 8u / C : 1u);
        double sum = 0.0;
#pragma unroll
        for (uint32_t q = 0; q < (uint32_t)C; ++q) {
            const float4 x = from[(q + turn) & (uint32_t)(C - 1)];
            sum += (double)x.x;
            sum += (double)x.y;
            sum += (double)x.z;
            sum += (double)x.w;
        }
        // (blocks behind the last group of chunks that holds elements have not been written)
        if constexpr (!FULL) sum = BLOCK * lane < my_len ? sum : 0.0;
        const double incl = wave_inclusive_scan_f64(sum);
        my.prefix[64u * part + lane] = incl - sum;  // within the wavefront's positions, for the time being
        if (lane == 63u) my.wave_sum[part] = incl;

        // may the fp64 sums round?  (small elements sit in the bins next to zero: see any_tiny_element)
        constexpr uint32_t SAFE = safe_binades((uint32_t)Bucket::D);
        const uint32_t biased = mag_max >> 23;
        if (biased > SAFE) {
            const uint32_t mag_safe = (biased - SAFE) << 23;
            const uint32_t near = magnitude_bin<(int)HALF>(__uint_as_float(mag_safe), bins_of) + 1u;
            const char* grouped = reinterpret_cast<const char*>(my.grouped);
            const uint32_t last = my.bin_start[HALF + near];
            bool tiny = false;
            for (uint32_t p = my.bin_start[HALF - near] + 4u * (64u * part + lane); p < last; p += 4u * 64u * W) {
                const uint32_t magnitude = *reinterpret_cast<const uint32_t*>(grouped + p) & 0x7FFFFFFFu;
                tiny = tiny || (magnitude != 0u && magnitude < mag_safe);
            }
            if (tiny) my.tiny = 1u;
        }
        // the level records of the ends: the bottom level is only ever the left end of a solve, the top level the right end
        if (part == 0u && lane < (uint32_t)S) {
            const bool top = lane == (uint32_t)(S - 1);
            GroupLevel end;
            end.value = top ? high : low;
            end.count_lt = end.count_le = (uint16_t)(top ? len : 0u);
            end.sum_lt = end.sum_le = 0.0;  // (the top level's follows below)
            end.rank = 0u;
            my.level[lane] = end;
            my.bins = bins_of;
        }
    }
    __syncthreads();

    // ---- the levels of all buckets, on one wavefront (another one from workgroup to workgroup: a CU's wavefronts are dealt
    //      to its SIMDs in order) -----------------------------------------------------------------------------------------
    // The random numbers, a third of the encoder, do not depend on the levels: the wavefronts that wait make theirs meanwhile, and all (with two
    // wavefronts in the workgroup: half) of those of the one that solves, which takes them through LDS.  Eight levels, two sweeps, 143.7 M values in buckets
    // of 4096 310 -> 292 us (each its own, the solving wavefront behind the others: 300); four levels, 25.6 M in buckets of 2048 51.5 -> 45.8 (49.1).
    // None are made for chunks without elements: with them four levels, two sweeps, 1628 buckets of 3072, whose second wavefronts hold half, took 20.4 us, each
    // its own 19.1, now 19.7.
    const EncodeRange range = one_range<BITS>(my_len, begin + first, seed, index_offset, codes32);
    constexpr uint32_t HELPERS = (uint32_t)(NB * W) - 1u;
    constexpr int SHARE = HELPERS == 3u ? (C + 2) / 3 : C / 2;                        // chunks helper, helper + HELPERS, ... of them
    constexpr int HANDED = (int)HELPERS * SHARE < C ? (int)HELPERS * SHARE : C;       // it makes the others itself
    DrawsAhead<C> draws;
    DrawsAhead<SHARE> share;
    const uint32_t solver = (blockIdx.x * 0x9E3779B1u >> 16) % (HELPERS + 1u), helper = (wave - solver - 1u) & HELPERS;
    const bool solves = wave == solver;
    if (solves) {
        __builtin_amdgcn_s_setprio(kSolving);
        if constexpr (W == 2) {
            // the second wavefronts' prefixes count from their own first position
            double before[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) before[b] = lds.bucket[b].wave_sum[0] + lds.bucket[b].prefix[64u + lane];
#pragma unroll
            for (int b = 0; b < NB; ++b) lds.bucket[b].prefix[64u + lane] = before[b];
        }
        constexpr uint32_t G = 16;
        constexpr uint32_t LANES = 64u / NB;  // of a bucket
        static_assert(LANES >= pool_chains(S) * G, "a group per bucket and chain");
        Bucket& b = lds.bucket[lane / LANES];
        double total = b.wave_sum[0];
        if constexpr (W == 2) total += b.wave_sum[1];
        b.level[S - 1].sum_le = total;  // (the same from all lanes of the bucket)
        wave_lds_sync();
        const uint32_t of_bucket = blockIdx.x * (uint32_t)NB + lane / LANES;
        uint32_t its_len = (uint32_t)Bucket::D;
        if constexpr (!FULL) {
            const size_t at = (size_t)of_bucket * bucket_size;
            its_len = of_bucket >= num_buckets ? 0u : n - at < bucket_size ? (uint32_t)(n - at) : bucket_size;
        }
        const uint32_t at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) Bucket*)&b;
        const uint32_t limb = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned long long*)lds.exact_limb;
        group_solve_levels_direct<pool_chains(S), S, Bucket>(b.view(lds.exact_limb, its_len), __builtin_fabs(total) < __builtin_inf(), sweeps, lane,
                                                          [&](uint32_t entry) __attribute__((always_inline)) {
                                                              return uniform_u32(pool_solve_general<Bucket>(at, limb, its_len, entry, lane)) != 0u;
                                                          });
        __builtin_amdgcn_s_setprio(kAtWork);
    } else {
        __builtin_amdgcn_s_setprio(kAhead);
        draws.template make<OneRange, !FULL>(range);
        const uint32_t its_bucket = blockIdx.x * (uint32_t)NB + solver / (uint32_t)W, its_first = PER_WAVE * (solver % (uint32_t)W);
        // (as many as a whole bucket has, and none behind those that are handed over)
        const uint32_t its_len = FULL ? 256u * HANDED : __builtin_elementwise_sub_sat(bucket_size, its_first);
        share.template make<OneRange, (!FULL || HANDED < (int)HELPERS * SHARE), (int)HELPERS>(
            one_range<BITS>(its_len < 256u * HANDED ? its_len : 256u * HANDED, (size_t)its_bucket * bucket_size + its_first, seed, index_offset, codes32),
            helper);
        __builtin_amdgcn_s_setprio(kAtWork);
    }
    __syncthreads();
    {
        // (the grouped values are no longer read; the encoder's tables lie at their beginning)
        static_assert(Bucket::D >= 256 * HANDED && (S <= kScaledWidthLevels || Bucket::D > 256 * HANDED), "place for both");
        floatx4* place = reinterpret_cast<floatx4*>(lds.bucket[0].grouped + (Bucket::D - 256 * HANDED)) + lane;
        if (!solves) {
#pragma unroll
            for (int t = 0; t < SHARE; ++t) {
                const uint32_t c = helper + HELPERS * (uint32_t)t;
                if (c < (uint32_t)HANDED) place[64u * c] = floatx4{share.draw[t][0], share.draw[t][1], share.draw[t][2], share.draw[t][3]};
            }
        }
        __syncthreads();
        if (solves) {
            draws.template make<OneRange, !FULL, 1, HANDED>(range);
#pragma unroll
            for (int c = 0; c < HANDED; ++c) {
                const floatx4 x = place[64 * c];
                draws.draw[c][0] = x.x; draws.draw[c][1] = x.y; draws.draw[c][2] = x.z; draws.draw[c][3] = x.w;
            }
        }
    }

    float lv[S];
#pragma unroll
    for (int k = 0; k < S; ++k) lv[k] = my.level[k].value;
    if constexpr (!(C < 8 && S == 4)) {  // (kept through the solves but for the kernel that has 96 registers: three would go to scratch memory)
        lv[0] = low;
        lv[S - 1] = high;
    }
    if (part == 0u && exists) {
        float mine = lv[0];
#pragma unroll
        for (int k = 1; k < S; ++k) mine = lane == (uint32_t)k ? lv[k] : mine;
        if (lane < (uint32_t)S) levels[(size_t)bucket * S + lane] = mine;
    }
    encode_all<OneRange, C, S, BITS, FULL ? Fill::kAll : Fill::kRagged>(v, lv, range, ReloadFromMemory{g + first, my_len, limit},
                                                                        encoder_table<S, true>(my.grouped, part), draws);
}

// (Five wavefronts per SIMD with four levels up to 1024 elements: 12290 buckets of 768, two sweeps, four 36 us, five 30.)
template <int W, int C, int S, int BITS>
__global__ __launch_bounds__(pool_buckets(W, S) * W * kWave) __attribute__((amdgpu_waves_per_eu(C == 8 ? 4 : S == 4 ? 5 : 1))) void orq_pool_kernel(
    const float* __restrict__ grad, size_t n, uint32_t bucket_size, uint32_t sweeps, float clip, uint32_t num_buckets, uint64_t seed,
    uint64_t index_offset, float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    __shared__ __attribute__((aligned(16))) PoolLds<W, C, S> lds;
    static_assert(sizeof(lds) <= 65536, "an LDS address in 16 bits");
    static_assert(C != 8 || sizeof(lds) <= (size_t)W * pool_buckets(W, S) * 10240, "16 wavefronts in a CU");
    constexpr uint32_t D = PoolBucket<W, C, S>::D;
    if (bucket_size == D && ((size_t)blockIdx.x + 1u) * (pool_buckets(W, S) * D) <= n)
        orq_pool_group<W, C, S, BITS, true>(lds, grad, n, bucket_size, sweeps, clip, num_buckets, seed, index_offset, levels, codes32);
    else
        orq_pool_group<W, C, S, BITS, false>(lds, grad, n, bucket_size, sweeps, clip, num_buckets, seed, index_offset, levels, codes32);
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------
template <int W, int C, int S, int BITS>
void launch_orq_pool(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    constexpr int NB = pool_buckets(W, S);
    launch_kernel((orq_pool_kernel<W, C, S, BITS>), dim3((nb + NB - 1) / NB), dim3(NB * W * kWave), st, g, n, p->bucket_size, p->level_iters,
                  p->clip_factor, nb, p->seed, p->index_offset, lv, static_cast<uint32_t*>(codes));
}

}  // namespace ogq
#endif  // OGQ_POOL_KERNELS_H
