// Internal header of libogq: the random-rounding quantize kernel for large buckets whose rule places one interior level
// (ORQ-3, Linear-3).  Included by rounding_part.hip after rounding_kernels.h, whose binning, exact sums and encoder it
// uses.  Compile with -ffp-contract=off.
#ifndef OGQ_GATHER_KERNELS_H
#define OGQ_GATHER_KERNELS_H

#include "rounding_kernels.h"

namespace ogq {

// ----------------------------------------------------------------------------------------------
// Three levels, W wavefronts of a workgroup per bucket, wavefront w holding elements [256 C w, 256 C (w + 1)) in the
// register layout of orq_bucket.
//
// The one interior level is the element of a single rank, and the rank follows from the bucket's total alone (ORQ-3) or
// from its length (Linear-3).  So the bucket is not grouped in LDS: a histogram of finer bins than orq_team_kernel's tells
// which bin holds the rank, the wavefronts collect that bin's few elements from their registers, and one of them picks.
// What bounds orq_team_kernel at 32768 elements is the LDS of the grouped bucket, 143 KB: one workgroup of 8
// wavefronts per CU, whose phases nothing overlaps (ORQ-3, 25.6 M values: 75 us with the vector units busy 46 % of the
// time).  Here a bucket takes at most 22 KB and the registers decide: 16 wavefronts of 128 registers fill a CU.
//
// Bound by the phases of a bucket that all its wavefronts go through together.  Two buckets share a CU: above 16384 elements as
// 2 x 8 wavefronts that hold 64 elements per lane (103 of 128 registers); 16 wavefronts with 32 elements per lane fill a CU with one
// bucket, whose loads and barriers nothing overlaps.  It also matters that every pass makes what it needs of an element afresh
// (opaque_zero): kept from the histogram to the collection, v + 0 and the lane masks of the tests cost 64 registers.
// ORQ-3, 25.6 M values, orq_team_kernel -> 16 wavefronts, one bucket per CU -> now: buckets of 8192 42 -> 36 -> 36 us, 16384 59 -> 41 -> 35,
// 20480 105 -> 78 -> 60, 32768 75 -> 59 -> 45; 16 buckets of 32768 20 -> 14.  Workgroups that stay and fetch their next bucket into the free
// LDS meanwhile were slower (32768: 72 us).
// ----------------------------------------------------------------------------------------------
template <int W, int C>
struct GatherLds {
    static constexpr int D = 256 * C * W;
    // 16 binades per sign; 35 elements of a bucket of Gaussian values in the fullest bin
    static constexpr int B = D >= 32768 ? 4096 : D >= 16384 ? 2048 : 1024;
    static constexpr int SHIFT = D >= 32768 ? 16 : D >= 16384 ? 17 : 18;  // magnitude bits dropped
    static constexpr uint32_t LIST = 1024;
    uint32_t bin_count[B];
    uint32_t list[LIST];  // the wanted bin's elements but zeros (bit patterns), in any order
    uint32_t list_count;
    uint32_t wave_total[W];
    uint32_t wanted[3];  // bin that holds the rank, elements in front of it, elements in it
    float level;
    unsigned long long exact_limb[kExactLimbs];
    TeamSlot slots[2][W];
};

// floor(T) of the whole bucket in exact arithmetic, by all threads of the workgroup (see exact_floor_t): the elements are
// read once more from memory.  L < R are the bucket's extremes.
__device__ __forceinline__ uint32_t exact_floor_t_team(unsigned long long* limb, const float* g, uint32_t len,
                                                        float limit, uint32_t threads, float L, float R,
                                                        uint32_t guess)
{
    const uint32_t tid = threadIdx.x;
    __syncthreads();
    if (tid < (uint32_t)kExactLimbs) limb[tid] = 0ull;
    __syncthreads();
    for (uint32_t i = tid; i < len; i += threads) exact_add_shared(limb, clipped(g[i], limit) + 0.0f);
    __syncthreads();
    uint32_t lo = 0u, hi = len;  // m = 0 fits
    uint32_t probe = guess < len ? guess : len;
    if (probe == 0u) probe = hi > 0u ? 1u : 0u;
    for (int step = 0; lo < hi; ++step) {
        const uint32_t mid = step == 0 ? probe : (step == 1 && lo == probe && probe < hi) ? probe + 1u : lo + (hi - lo + 1u) / 2u;
        if (exact_not_negative(limb, L, -(long long)(len - mid), R, -(long long)mid)) lo = mid;
        else hi = mid - 1u;
    }
    return lo;
}

// The element of 1-based rank `rank` among the first `count` (more than 64 (K - 1), at most 64 K) of the list, as its key: quickselect by a wavefront that
// holds K keys per lane.  A pivot is an element that is still open; it leaves at least itself out of the next round, and only a rank beyond
// the list, which there is none of, leaves none open.
template <int K>
__device__ __forceinline__ uint32_t select_in_list(const uint32_t* list, uint32_t count, uint32_t rank, uint32_t lane)
{
    uint32_t mine[K];
    uint64_t open[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const uint32_t i = lane + 64u * (uint32_t)k;
        mine[k] = i < count ? float_to_key(__uint_as_float(list[i])) : 0xFFFFFFFFu;
        open[k] = __ballot(i < count);
    }
    for (;;) {
        uint32_t pivot = 0;
        bool found = false;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!found && open[k] != 0) {
                pivot = __builtin_amdgcn_readlane(mine[k], (uint32_t)__builtin_ctzll(open[k]));
                found = true;
            }
        }
        uint64_t below[K], not_above[K];
        uint32_t count_below = 0, count_not_above = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            below[k] = __ballot(mine[k] < pivot);
            not_above[k] = __ballot(mine[k] <= pivot);
            count_below += (uint32_t)__popcll(below[k]);
            count_not_above += (uint32_t)__popcll(not_above[k]);
        }
        if (!found || (count_below < rank && rank <= count_not_above)) return pivot;
        const bool lower = rank <= count_below;
#pragma unroll
        for (int k = 0; k < K; ++k) open[k] &= lower ? below[k] : ~not_above[k];
    }
}

template <int W, int C, int BITS, bool FULL, int RULE>
__device__ __forceinline__ void orq_gather_bucket(GatherLds<W, C>& lds, const float* __restrict__ g, uint32_t len, size_t begin,
                                                  uint32_t bucket, float clip, uint64_t seed, uint64_t index_offset,
                                                  float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    static_assert(RULE == kOptimal || RULE == kLinear, "rules with one interior level");
    using Lds = GatherLds<W, C>;
    constexpr uint32_t PER_WAVE = 256u * C, THREADS = 64u * W;
    constexpr uint32_t B = Lds::B, HALF = B / 2;
    constexpr int SHIFT = Lds::SHIFT;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t wave = uniform_u32(tid >> 6);
    const uint32_t first = PER_WAVE * wave;
    const uint32_t my_len = len > first ? (len - first < PER_WAVE ? len - first : PER_WAVE) : 0u;
    WaveTeam<W> team{lds.slots, wave, 0u};

    for (uint32_t i = tid; i < B; i += THREADS) lds.bin_count[i] = 0u;
    if (tid == 0u) lds.list_count = 0u;
    float v[C][4];
    load_range<C, FULL>(v, g, first, len, my_len, lane);

    float limit = __uint_as_float(0x7F800000u);  // clipping threshold
    if (clip > 0.0f) {  // the same for every thread of the grid
        float(&flat)[4 * C] = reinterpret_cast<float(&)[4 * C]>(v);
        uint32_t here = lane;
        limit = clip_in_registers<4 * C>(
            flat, len, clip, [&](int j) { return FULL || (64u * (j & ~3) + 4u * here + (j & 3) < my_len); },
            [&](double& x, double& y) __attribute__((always_inline)) {
                if constexpr (!FULL) asm volatile("" : "+v"(here));  // (see set_padding)
                x = wave_sum(x);
                y = wave_sum(y);
                team.sums(x, y);
            });
        if constexpr (!FULL) set_padding<C>(v, my_len, lane);
    }

    // ---- extremes and (ORQ) total of the bucket ---------------------------------------------------------
    float low, high;
    uint32_t unused_zeros;
    lane_extremes<C, false>(v, low, high, unused_zeros);
    double part = 0.0;
    if constexpr (RULE == kOptimal) {
        for_each_chunk<C, FULL>(my_len, [&](int c, auto all) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                part += (double)(decltype(all)::value || 256u * c + 4u * lane + k < my_len ? v[c][k] : 0.0f);
        });
    }
    wave_extremes(low, high);
    double total = 0.0;
    {
        const TeamSlot* s = team.exchange(RULE == kOptimal ? wave_sum(part) : 0.0, __float_as_uint(low), __float_as_uint(high));
#pragma unroll
        for (int w = 0; w < W; ++w) {
            low = fminf(low, __uint_as_float(s[w].a));
            high = fmaxf(high, __uint_as_float(s[w].b));
            total += s[w].sum;
        }
    }
    low = uniform_f32(low + 0.0f);  // -0 -> +0
    high = uniform_f32(high + 0.0f);
    const uint32_t mag_max = umax32(__float_as_uint(low) & 0x7FFFFFFFu, __float_as_uint(high) & 0x7FFFFFFFu);
    const uint32_t t_low = __builtin_elementwise_sub_sat(mag_max >> SHIFT, HALF - 1u);

    // ---- histogram (the exchange's barrier lies behind the zeroing) --------------------------------------
    const float zero = opaque_zero();
    for_each_chunk<C, FULL>(my_len, [&](int c, auto all) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool valid = decltype(all)::value || (256u * c + 4u * lane + k < my_len);
            // (padding adds 0 to one bin per lane: no branch)
            const uint32_t bin = value_bin<(int)HALF, SHIFT>(v[c][k] + zero, t_low);
            atomicAdd(&lds.bin_count[valid ? bin : lane], valid ? 1u : 0u);
        }
    });
    __syncthreads();

    // ---- rank of the level ------------------------------------------------------------------------------
    uint32_t rank;  // 1-based
    bool ordered = true;
    if constexpr (RULE == kLinear) {
        rank = 1u + (len - 1u) / 2u;
    } else {
        ordered = low < high;
        // S = sum (v - L) over the bucket, T = S / (R - L), level = element of rank len - floor(T)
        const double Ssum = total - (double)low * (double)len, width = (double)high - (double)low;
        // The sums may round unless the bins below the safe range are empty (see any_tiny_element; zeros count as small
        // here: the bound then only sends a solve to the exact sums that the others would not need them for).
        constexpr uint32_t SAFE = safe_binades(Lds::D);
        const uint32_t biased = mag_max >> 23;
        uint32_t small = 0u;
        if (biased > SAFE) {
            const uint32_t t_safe = ((biased - SAFE) << 23) >> SHIFT;
            const uint32_t near = umin32(t_safe > t_low ? t_safe - t_low : 1u, HALF);
            for (uint32_t i = lane; i < 2u * near; i += kWave) small |= lds.bin_count[HALF - near + i];
        }
        const double bound = __ballot(small != 0u) != 0 ? sum_error_bound_of(mag_max, Lds::D) : 0.0;
        double m;
        const bool decided = floor_t_from_sums(Ssum, width, bound, m);
        if (ordered && !decided)  // (the same for all threads: they hold the same sums)
            m = (double)exact_floor_t_team(lds.exact_limb, g, len, limit, THREADS, low, high, (uint32_t)m);
        const uint32_t below = uniform_u32((uint32_t)fmin(m, 65536.0));
        rank = below >= len ? 1u : len - below;
    }

    // ---- the bin that holds the rank: thread t owns bins [t PER, (t + 1) PER) ---------------------------------
    {
        constexpr uint32_t PER = B / THREADS;
        static_assert(PER >= 4 && PER % 4 == 0, "16-byte reads");
        uint32_t count[PER], mine = 0;
#pragma unroll
        for (uint32_t q = 0; q < PER / 4u; ++q) {
            const uint4 x = reinterpret_cast<const uint4*>(lds.bin_count)[tid * (PER / 4u) + q];
            count[4 * q] = x.x; count[4 * q + 1] = x.y; count[4 * q + 2] = x.z; count[4 * q + 3] = x.w;
            mine += (x.x + x.y) + (x.z + x.w);
        }
        const uint32_t incl = wave_inclusive_scan_u32(mine);
        if (lane == 63u) lds.wave_total[wave] = incl;
        __syncthreads();
        uint32_t before = incl - mine;
#pragma unroll
        for (int w = 0; w < W; ++w) before += (uint32_t)w < wave ? lds.wave_total[w] : 0u;
        if (before < rank && rank <= before + mine) {  // one thread of the workgroup
            // (in a straight line: read again bin by bin, every wavefront waits for up to PER trips to LDS)
            uint32_t at = 0, front = before, in_it = count[0];
#pragma unroll
            for (uint32_t i = 1; i < PER; ++i) {
                before += count[i - 1];
                const bool further = before < rank;
                at = further ? i : at;
                front = further ? before : front;
                in_it = further ? count[i] : in_it;
            }
            lds.wanted[0] = tid * PER + at;
            lds.wanted[1] = front;
            lds.wanted[2] = in_it;
        }
        __syncthreads();
    }
    const uint32_t bin = uniform_u32(lds.wanted[0]), in_front = uniform_u32(lds.wanted[1]);
    uint32_t count = uniform_u32(lds.wanted[2]), in_bin = rank - in_front;  // in_bin: 1-based

    // ---- collect the bin's elements: those whose bit pattern lies in [from, from + range) -----------------
    // Zeros, which sparse gradients have thousands of, are left out: they are the first elements of their bin, and as many as the
    // list then lacks (half of the values zero, 300 buckets of 32768: 139 -> 43 us).
    const bool negative = bin < HALF;
    const uint32_t u = negative ? HALF - 1u - bin : bin - HALF;
    const uint32_t sign = negative ? 0x80000000u : 0u;
    const uint32_t from = sign | (u == 0u ? 1u : (t_low + u) << SHIFT);
    const uint32_t range = (u == HALF - 1u ? sign + 0x80000000u : sign | ((t_low + u + 1u) << SHIFT)) - from;
    uint32_t smallest = 0xFFFFFFFFu, largest = 0u;
    // (-0 need not be turned into +0 first: neither is in any range.  One branch for four elements, of which few are wanted,
    // and the bin of the rank in a straight line: 25.6 M values in buckets of 32768 43.6 -> 42.4 us)
    for_each_chunk<C, FULL>(my_len, [&](int c, auto all) __attribute__((always_inline)) {
        bool wanted[4], some = false;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool valid = decltype(all)::value || (256u * c + 4u * lane + k < my_len);
            wanted[k] = valid && __float_as_uint(v[c][k]) - from < range;
            some = some || wanted[k];
        }
        if (__ballot(some) != 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (wanted[k]) {
                    const float x = v[c][k];
                    const uint32_t at = atomicAdd(&lds.list_count, 1u);
                    if (at < Lds::LIST) lds.list[at] = __float_as_uint(x);
                    smallest = umin32(smallest, float_to_key(x));
                    largest = umax32(largest, float_to_key(x));
                }
            }
        }
    });
    uint32_t key;
    if (bin == HALF) {
        __syncthreads();
        const uint32_t others = uniform_u32(lds.list_count), zeros = count - others;
        count = in_bin <= zeros ? 0u : others;
        in_bin -= zeros;
    }
    if (count == 0u) {
        key = float_to_key(0.0f);
    } else if (count <= 64u) {
        __syncthreads();
        const uint32_t mine = lane < count ? float_to_key(__uint_as_float(lds.list[lane])) : 0xFFFFFFFFu;
        uint32_t not_above;
        select_rank(mine, count, in_bin, ~0ull >> (64u - count), key, not_above);
    } else if (count <= 256u) {
        // The bins next to zero hold all that is more than 16 binades below the largest magnitude, some 70 elements of a mixture of scales at
        // 32768, and the level is often found there.  25.6 M such values in buckets of 32768 46.6 us with the bisection below, 41.4 with this
        // (one card; 256 buckets 23.9 and 17.8).
        __syncthreads();
        key = count <= 128u ? select_in_list<2>(lds.list, count, in_bin, lane) : select_in_list<4>(lds.list, count, in_bin, lane);
    } else {
        // A more crowded bin: bisection over the bits in which its smallest and largest key differ (none when all its values
        // are equal), on the list, or where that is too short on the registers of all wavefronts.
        smallest = wave_min_u32(smallest);
        largest = wave_max_u32(largest);
        const TeamSlot* s = team.exchange(0.0, smallest, largest);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            smallest = umin32(smallest, s[w].a);
            largest = umax32(largest, s[w].b);
        }
        smallest = uniform_u32(smallest);
        const uint32_t differing = uniform_u32(smallest ^ largest);
        key = smallest;
        if (differing != 0u) {
            const int top = 31 - __builtin_clz(differing);
            key = top == 31 ? 0u : smallest & ~((2u << top) - 1u);
#pragma unroll 1
            for (int bit = top; bit >= 0; --bit) {
                const uint32_t candidate = key | (1u << bit);
                uint32_t below = 0;
                if (count <= Lds::LIST) {
                    for (uint32_t i = lane; i < count; i += kWave)
                        below += float_to_key(__uint_as_float(lds.list[i])) < candidate ? 1u : 0u;
                    below = wave_sum_u32(below);
                } else {
                    const float once_more = opaque_zero();
                    for_each_chunk<C, FULL>(my_len, [&](int c, auto all) __attribute__((always_inline)) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const bool valid = decltype(all)::value || (256u * c + 4u * lane + k < my_len);
                            const float x = v[c][k] + once_more;
                            below += valid && __float_as_uint(x) - from < range && float_to_key(x) < candidate ? 1u : 0u;
                        }
                    });
                    double unused = 0.0;
                    below = wave_sum_u32(below);
                    team.sum_and_count(unused, below);
                }
                if (uniform_u32(below) < in_bin) key = candidate;
            }
        }
    }
    const float picked = key_to_float(key);
    const float lv[3] = {low, ordered && !(picked < low) ? picked : low, high};
    if (tid < 3u) levels[(size_t)bucket * 3 + tid] = tid == 0u ? lv[0] : tid == 1u ? lv[1] : lv[2];

    orq_encode<C, 3, BITS, FULL>(v, lv, my_len, begin + first, seed, index_offset, codes32, ReloadFromMemory{g + first, my_len, limit});
}

template <int W, int C, int BITS, int RULE>
__global__ __launch_bounds__(W* kWave) __attribute__((amdgpu_waves_per_eu(4))) void orq_gather_kernel(
    const float* __restrict__ grad, size_t n, uint32_t bucket_size, float clip, uint32_t num_buckets, uint64_t seed,
    uint64_t index_offset, float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    __shared__ GatherLds<W, C> lds;
    const uint32_t bucket = blockIdx.x;
    if (bucket >= num_buckets) return;
    const size_t begin = (size_t)bucket * bucket_size;
    const size_t rest = n - begin;
    const uint32_t len = rest < bucket_size ? (uint32_t)rest : bucket_size;
    const float* g = grad + begin;
    if (len == (uint32_t)GatherLds<W, C>::D)
        orq_gather_bucket<W, C, BITS, true, RULE>(lds, g, len, begin, bucket, clip, seed, index_offset, levels, codes32);
    else
        orq_gather_bucket<W, C, BITS, false, RULE>(lds, g, len, begin, bucket, clip, seed, index_offset, levels, codes32);
}

// Whether the scheme is one of this kernel's, and if so the launch.
template <int W, int C>
bool launch_gather(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if (p->bits != 2 || (p->scheme != OGQ_ORQ_PAPER && p->scheme != OGQ_LINEAR)) return false;
    launch_kernel(p->scheme == OGQ_ORQ_PAPER ? orq_gather_kernel<W, C, 2, kOptimal> : orq_gather_kernel<W, C, 2, kLinear>, dim3(nb),
                  dim3(W * kWave), st, g, n, p->bucket_size, p->clip_factor, nb, p->seed, p->index_offset, lv,
                  static_cast<uint32_t*>(codes));
    return true;
}

}  // namespace ogq
#endif  // OGQ_GATHER_KERNELS_H
