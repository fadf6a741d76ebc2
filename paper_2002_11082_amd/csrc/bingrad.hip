// libogq, BinGrad-b and Scaled SignSGD quantize kernels (Section 3.2 of arXiv 2002.11082) for MI355X (gfx950).
// Compile with -ffp-contract=off.
#include "device_common.h"
#include "launch.h"

namespace ogq {

// x unchanged, but opaque to the optimizer: what is derived from it is computed again instead of kept in registers.
__device__ __forceinline__ float reread(float x)
{
    asm volatile("" : "+v"(x));
    return x;
}

// ----------------------------------------------------------------------------------------------
// BinGrad-b quantize.  Lane l register j holds bucket element 64*j + l, so a ballot over
// register j is the packed code word j of the bucket.
// ----------------------------------------------------------------------------------------------
// E registers per lane; FULL: every register of this wavefront holds a bucket element.  g, len, levels2
// and words belong to the whole bucket, of which this wavefront holds the 64*E elements from `first_element` on;
// the wavefront with first_element == 0 writes the levels.  SIGN: Scaled SignSGD instead (first equation of
// Section 3.2): levels -m, +m with m the mean magnitude of the bucket, index = (v >= 0).
//
// Where elements are missing, padding holds 0, which adds nothing to a sum, its
// bits are cleared when the words are stored, and where 0 lies below the threshold its number is taken off the count.
// (With bounds tests per element instead: one bucket of 20480 elements
// 7.6 us, of 3008 with two updates 6.9, now 6.9, 5.3; 25.6 M values in buckets of 1344 34 -> 24 us.)
template <int E, bool FULL, bool CLIP, bool SIGN, class Team>
__device__ __forceinline__ void bingrad_bucket(Team team, uint32_t first_element, const float* __restrict__ g,
                                               uint32_t len, uint32_t iters, float clip, float* __restrict__ levels2,
                                               uint64_t* __restrict__ words)
{
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t first = first_element + lane;
    float v[E];
    if constexpr (FULL) {
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = __builtin_nontemporal_load(g + first + 64u * j);  // read once: bypass the caches
    } else if (first_element >= len) {
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = 0.0f;
    } else {
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const uint32_t e = first + 64u * j;
            v[j] = __builtin_nontemporal_load(g + (e < len ? e : 0u));
        }
        uint32_t here = first;
        if constexpr (E > 16) asm volatile("" : "+v"(here));  // (the loads' lane masks would not fit the scalar registers)
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = here + 64u * j < len ? v[j] : 0.0f;
    }
    const uint32_t padding = 64u * E * Team::kSize - len;
    if constexpr (CLIP) {
        uint32_t here = first;
        const auto bucket_sums = [&](double& x, double& y) {
            if constexpr (!FULL && E > 16) asm volatile("" : "+v"(here));  // (the first pass's lane masks would not fit the scalar registers)
            x = wave_sum(x);
            y = wave_sum(y);
            team.sums(x, y);
        };
        clip_in_registers<E>(v, len, clip, [&](int j) { return FULL || here + 64u * j < len; }, bucket_sums);
    }

    double part = 0.0;
    float mag = 0.0f;
#pragma unroll
    for (int j = 0; j < E; ++j) {
        part += (double)(SIGN ? fabsf(v[j]) : v[j]);
        mag = fmaxf(mag, fabsf(v[j]));
    }
    double total = wave_sum(part);
    float largest = wave_max(mag);
    team.sum_and_max(total, largest);
    float b0 = (float)(total / (double)len);  // threshold starts at the bucket mean
    // The upper sum is taken as total - lower sum.  Both are fp64 sums of the bucket's n <= 32768 fp32 values
    // (error below 2^-53 * n^2 * max|v| each, and exact for any bucket whose non-zero values span at most
    // 28 - log2(n) binades: 17 for 2048 elements, 13 for 32768), so the difference is trusted unless it is tiny
    // against the largest element; such a bucket sums its upper side directly.
    const float trust_above = 1e-3f * largest;

    double b_lo = 0.0, b_hi = 0.0;
    uint32_t word_lo = 0, word_hi = 0;  // lane j ends up holding packed word j of this wavefront's elements
    uint32_t prev_n_lo = 0xFFFFFFFFu;
    if constexpr (SIGN) {
#pragma unroll
        for (int j = 0; j < E; ++j) {
            const uint64_t hi_mask = ~__ballot(v[j] < 0.0f);
            word_lo = writelane(word_lo, (uint32_t)hi_mask, j);
            word_hi = writelane(word_hi, (uint32_t)(hi_mask >> 32), j);
        }
        b_hi = total / (double)len;
        b_lo = -b_hi;
    } else
    for (uint32_t it = 0;; ++it) {
        double s_lo = 0.0;
        uint32_t below = 0;
#pragma unroll
        for (int j = 0; j < E; ++j) {
            // (with 64 registers of data the fp64 copies the compiler would keep from the first pass do not fit)
            const float x = E > 32 ? reread(v[j]) : v[j];
            const bool lo = x < b0;
            const uint64_t hi_mask = ~__ballot(lo);
            below += lo ? 1u : 0u;
            s_lo += (double)(lo ? x : 0.0f);
            word_lo = writelane(word_lo, (uint32_t)hi_mask, j);
            word_hi = writelane(word_hi, (uint32_t)(hi_mask >> 32), j);
        }
        s_lo = wave_sum(s_lo);
        uint32_t n_lo = wave_sum_u32(below);
        team.sum_and_count(s_lo, n_lo);
        if ((!FULL || Team::kSize > 1) && 0.0f < b0) n_lo -= padding;
        double s_hi = total - s_lo;
        if (!(fabs(s_hi) >= (double)trust_above)) {
            double direct = 0.0;
#pragma unroll
            for (int j = 0; j < E; ++j) {
                direct += (double)(!(v[j] < b0) ? v[j] : 0.0f);
            }
            s_hi = team.sum(wave_sum(direct));
        }
        const uint32_t n_hi = len - n_lo;
        {
            // both conditional means with one division sequence: lane 0 divides the lower side, the
            // other lanes the upper side
            const double num = lane == 0 ? s_lo : s_hi;
            const uint32_t den = lane == 0 ? n_lo : n_hi;
            const double quot = num / (double)(den > 0 ? den : 1u);
            if (n_lo > 0) b_lo = readlane_f64(quot, 0);
            if (n_hi > 0) b_hi = readlane_f64(quot, 1);
        }
        if (n_lo == 0) b_lo = b_hi;  // constant bucket: both levels equal
        if (n_hi == 0) b_hi = b_lo;
        // Further threshold updates are identities once the partition repeats.
        if (it == iters || n_lo == prev_n_lo) break;
        prev_n_lo = n_lo;
        b0 = (float)((b_lo + b_hi) * 0.5);
    }

    if (lane == 0 && first_element == 0) {
        levels2[0] = (float)b_lo;
        levels2[1] = (float)b_hi;
    }
    const uint32_t word = first_element / 64u + lane;
    if constexpr (FULL) {
        if (lane < (uint32_t)E) words[word] = ((uint64_t)word_hi << 32) | word_lo;
    } else if (lane < (uint32_t)E && 64u * word < len) {
        const uint32_t left = len - 64u * word;
        const uint64_t valid = left < 64u ? (1ull << left) - 1ull : ~0ull;
        words[word] = (((uint64_t)word_hi << 32) | word_lo) & valid;
    }
}

constexpr int kBinGradWaves = 2;  // buckets per workgroup

// At most 4 waves per SIMD and small workgroups: with more, all resident waves load and then
// compute in lock-step and the tail of a launch that is only ~1.5 waves of workgroups deep is not
// overlapped.
template <int E, bool CLIP, bool SIGN>
__global__ __launch_bounds__(kWave* kBinGradWaves) __attribute__((amdgpu_waves_per_eu(4, 4))) void bingrad_quantize_kernel(
    const float* __restrict__ grad, size_t n, uint32_t bucket_size, uint32_t iters, float clip, uint32_t num_buckets,
    float* __restrict__ levels, uint64_t* __restrict__ codes)
{
    const uint32_t bucket = uniform_u32(blockIdx.x * kBinGradWaves + (threadIdx.x >> 6));
    if (bucket >= num_buckets) return;
    const size_t begin = (size_t)bucket * bucket_size;
    const size_t rest = n - begin;
    const uint32_t len = rest < bucket_size ? (uint32_t)rest : bucket_size;
    const float* g = grad + begin;
    float* lv = levels + (size_t)bucket * 2;
    uint64_t* w = codes + begin / 64;
    if (len == 64u * E) bingrad_bucket<E, true, CLIP, SIGN>(OneWave{}, 0u, g, len, iters, clip, lv, w);
    else bingrad_bucket<E, false, CLIP, SIGN>(OneWave{}, 0u, g, len, iters, clip, lv, w);
}

// Buckets of more than 2048 elements: the W = 2, 4, 8 or 16 wavefronts of a workgroup hold one bucket, E = 32
// registers per lane each as for a 2048-element bucket, and combine their sums and counts through LDS.  Above
// 8192 elements E = 64 (without clipping), so that a workgroup is at most 8 wavefronts and two buckets share a
// compute unit: the loads of one overlap the passes of the other.
template <int W, int E, bool CLIP, bool SIGN>
__global__ __launch_bounds__(W* kWave) __attribute__((amdgpu_waves_per_eu(4, 4))) void bingrad_team_kernel(
    const float* __restrict__ grad, size_t n, uint32_t bucket_size, uint32_t iters, float clip, uint32_t num_buckets,
    float* __restrict__ levels, uint64_t* __restrict__ codes)
{
    __shared__ TeamSlot slots[2][W];
    const uint32_t bucket = blockIdx.x;
    if (bucket >= num_buckets) return;
    const size_t begin = (size_t)bucket * bucket_size;
    const size_t rest = n - begin;
    const uint32_t len = rest < bucket_size ? (uint32_t)rest : bucket_size;
    const float* g = grad + begin;
    float* lv = levels + (size_t)bucket * 2;
    uint64_t* w = codes + begin / 64;
    const uint32_t wave = uniform_u32(threadIdx.x >> 6);
    const WaveTeam<W> team{slots, wave, 0u};
    constexpr uint32_t PER_WAVE = 64u * E;
    // Both variants reach the same combines in the same order (every branch around one depends on combined values only).
    if (PER_WAVE * (wave + 1u) <= len) bingrad_bucket<E, true, CLIP, SIGN>(team, PER_WAVE * wave, g, len, iters, clip, lv, w);
    else bingrad_bucket<E, false, CLIP, SIGN>(team, PER_WAVE * wave, g, len, iters, clip, lv, w);
}

// ----------------------------------------------------------------------------------------------
// BinGrad-b for buckets of up to 1024 elements: one wavefront quantizes NB = 32 / E whole buckets of 64 E
// elements at once (registers E*q .. E*q + E - 1 hold its bucket q in the layout above), so that a
// small bucket keeps as many loads in flight per wave as a 2048-element one and the per-bucket
// reductions and divisions are shared (25.6 M values, one bucket per wavefront -> several: buckets of 192 64 -> 20 us, of 320 43 -> 19,
// of 768 24.5 -> 18; with clipping of 64 160 -> 43, of 512 30 -> 20.5).  The NB partial results of a pass are reduced together: a
// step over lane bit 5, 4, 3, ... combines two partner lanes and halves the number of values a lane
// carries, the lanes with the bit clear keeping the even-numbered values and the others the
// odd-numbered ones.  When one value is left lane l holds the result of bucket q(l) = (l with its six
// bits reversed) mod TREE, and the remaining low lane bits are reduced as in wave_sum.  TREE is NB rounded up to a
// power of two; the places from NB on hold zeros.
// ----------------------------------------------------------------------------------------------
constexpr int kDppXor1From0 = 0xA0;  // quad_perm [0,0,2,2]: an odd lane takes the even lane below it

__device__ __forceinline__ double words_to_f64(uint32_t lo, uint32_t hi)
{
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// swap_halves: first = {a[0..31], b[0..31]}, second = {a[32..63], b[32..63]} (v_permlane32_swap).
// swap_rows: the same over pairs of 16-lane rows: first = {a.row0, b.row0, a.row2, b.row2},
// second = {a.row1, b.row1, a.row3, b.row3} (v_permlane16_swap).
__device__ __forceinline__ void swap_halves(float a, float b, float& first, float& second)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    first = __uint_as_float(r[0]);
    second = __uint_as_float(r[1]);
}

__device__ __forceinline__ void swap_halves(double a, double b, double& first, double& second)
{
    const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)ua, (uint32_t)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
    first = words_to_f64(lo[0], hi[0]);
    second = words_to_f64(lo[1], hi[1]);
}

__device__ __forceinline__ void swap_rows(float a, float b, float& first, float& second)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    first = __uint_as_float(r[0]);
    second = __uint_as_float(r[1]);
}

__device__ __forceinline__ void swap_rows(double a, double b, double& first, double& second)
{
    const uint64_t ua = (uint64_t)__double_as_longlong(a), ub = (uint64_t)__double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)ua, (uint32_t)ub, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(ua >> 32), (uint32_t)(ub >> 32), false, false);
    first = words_to_f64(lo[0], hi[0]);
    second = words_to_f64(lo[1], hi[1]);
}

template <int DIST>
__device__ __forceinline__ float lane_xor_val(float x, uint32_t lane)
{
    return __uint_as_float(lane_xor<DIST>(__float_as_uint(x), lane));
}

template <int DIST>
__device__ __forceinline__ double lane_xor_val(double x, uint32_t lane)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    return words_to_f64(lane_xor<DIST>((uint32_t)u, lane), lane_xor<DIST>((uint32_t)(u >> 32), lane));
}

template <int CTRL>
__device__ __forceinline__ float dpp_val(float x) { return dpp_f32<CTRL>(x); }
template <int CTRL>
__device__ __forceinline__ double dpp_val(double x) { return dpp_f64<CTRL>(x); }

// One reduction step over lane bit DIST (8, 4 or 2): lanes with the bit clear get a (+) a of the
// partner lane, the others b (+) b of the partner lane.
template <int DIST, class T, class Op>
__device__ __forceinline__ T fold_pair(T a, T b, uint32_t lane, Op op)
{
    const bool odd = (lane & (uint32_t)DIST) != 0;
    const T keep = odd ? b : a, send = odd ? a : b;
    return op(keep, lane_xor_val<DIST>(send, lane));
}

template <int Q>
struct BucketIndex {
    static constexpr int value = Q;
};

// Places FIRST .. FIRST + N - 1 of the wavefront, reduced depth first so that only one partial result
// per tree level is alive: leaf(BucketIndex<q>) yields this lane's partial value of bucket q < NB.
template <int N, int FIRST, int NB, class T, class Leaf, class Op>
__device__ __forceinline__ T reduce_bucket_tree(uint32_t lane, Leaf& leaf, Op op)
{
    if constexpr (FIRST >= NB) {
        return T(0);
    } else if constexpr (N == 1) {
        return leaf(BucketIndex<FIRST>{});
    } else {
        const T a = reduce_bucket_tree<N / 2, FIRST, NB, T>(lane, leaf, op);
        const T b = reduce_bucket_tree<N / 2, FIRST + N / 2, NB, T>(lane, leaf, op);
        if constexpr (N == 2) {
            T first, second;
            swap_halves(a, b, first, second);
            return op(first, second);
        } else if constexpr (N == 4) {
            T first, second;
            swap_rows(a, b, first, second);
            return op(first, second);
        } else if constexpr (N == 8) {
            return fold_pair<8>(a, b, lane, op);
        } else if constexpr (N == 16) {
            return fold_pair<4>(a, b, lane, op);
        } else {
            return fold_pair<2>(a, b, lane, op);
        }
    }
}

constexpr int tree_of(int nb)
{
    int tree = 2;
    while (tree < nb) tree *= 2;
    return tree;
}

template <int NB, class T, class Leaf, class Op>
__device__ __forceinline__ T reduce_buckets(uint32_t lane, Leaf leaf, Op op)
{
    static_assert(NB >= 2 && NB <= 32, "buckets per wavefront");
    constexpr int TREE = tree_of(NB);
    T r = reduce_bucket_tree<TREE, 0, NB, T>(lane, leaf, op);
    // the lane bits that select no bucket
    r = op(r, dpp_val<kDppXor1>(r));
    if constexpr (TREE <= 16) r = op(r, dpp_val<kDppXor2>(r));
    if constexpr (TREE <= 8) r = op(r, dpp_val<kDppHalfMirror>(r));
    if constexpr (TREE <= 4) r = op(r, dpp_val<kDppMirror>(r));
    if constexpr (TREE <= 2) {
        T first, second;
        swap_rows(r, r, first, second);
        r = op(first, second);
    }
    return r;
}

template <int NB, int Q = 0, class F>
__device__ __forceinline__ void for_each_bucket(F f)
{
    if constexpr (Q < NB) {
        f(BucketIndex<Q>{});
        for_each_bucket<NB, Q + 1>(f);
    }
}

constexpr uint32_t reverse6(uint32_t x)
{
    uint32_t r = 0;
    for (int b = 0; b < 6; ++b) r |= ((x >> b) & 1u) << (5 - b);
    return r;
}

constexpr int buckets_of_a_wavefront(int e) { return 32 / e; }

template <int E, bool CLIP, bool SIGN>
__global__ __launch_bounds__(kWave* kBinGradWaves) __attribute__((amdgpu_waves_per_eu(4, 4))) void bingrad_chunk_kernel(
    const float* __restrict__ grad, uint32_t num_chunks, uint32_t rest, uint32_t iters, float clip, float* __restrict__ levels,
    uint64_t* __restrict__ codes)
{
    constexpr int NB = buckets_of_a_wavefront(E), R = NB * E;
    constexpr uint32_t D = 64u * E;             // bucket size
    constexpr uint32_t CHUNK = 64u * R;         // elements of a wavefront
    constexpr uint32_t kFreeBits = 64u / tree_of(NB) - 1u;  // lane bits that select no place; bit 0 is always among them
    uint32_t chunk = uniform_u32(blockIdx.x * kBinGradWaves + (threadIdx.x >> 6));
    // The first wavefronts take the buckets behind the last whole chunk (`rest` elements), one each.
    const uint32_t rest_buckets = (rest + D - 1u) / D;
    if (chunk < rest_buckets) {
        const uint32_t bucket = chunk, len = rest - bucket * D < D ? rest - bucket * D : D;
        const size_t begin = (size_t)num_chunks * CHUNK + bucket * D;
        bingrad_bucket<E, false, CLIP, SIGN>(OneWave{}, 0u, grad + begin, len, iters, clip, levels + begin / D * 2, codes + begin / 64);
        return;
    }
    chunk -= rest_buckets;
    if (chunk >= num_chunks) return;
    const uint32_t lane = threadIdx.x & 63u;
    const float* g = grad + (size_t)chunk * CHUNK;
    float v[R];
#pragma unroll
    for (int j = 0; j < R; ++j) v[j] = __builtin_nontemporal_load(g + 64u * j + lane);

    const auto add = [](double a, double b) { return a + b; };
    const auto larger = [](float a, float b) { return fmaxf(a, b); };
    if constexpr (CLIP) {  // clip_in_registers, NB buckets at once
        const double sum = reduce_buckets<NB, double>(
            lane,
            [&](auto q) {
                double s = 0.0;
#pragma unroll
                for (int j = 0; j < E; ++j) s += (double)v[decltype(q)::value * E + j];
                return s;
            },
            add);
        const double squares = reduce_buckets<NB, double>(
            lane,
            [&](auto q) {
                double s = 0.0;
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    // (converted again: the fp64 copies of the first pass would not fit the registers)
                    const double x = (double)reread(v[decltype(q)::value * E + j]);
                    s = __builtin_fma(x, x, s);
                }
                return s;
            },
            add);
        bool cancels;
        double about_mean = squares_about_mean(sum, squares, (double)D, cancels);
        if (__builtin_expect(__ballot(cancels) != 0, 0)) {
            const double mean = sum / (double)D;
            const double again = reduce_buckets<NB, double>(
                lane,
                [&](auto q) {
                    constexpr int kQ = decltype(q)::value;
                    const double middle = readlane_f64(mean, (int)reverse6(kQ));
                    double s = 0.0;
#pragma unroll
                    for (int j = 0; j < E; ++j) {
                        const double dv = (double)reread(v[kQ * E + j]) - middle;
                        s += dv * dv;
                    }
                    return s;
                },
                add);
            about_mean = cancels ? again : about_mean;
        }
        const float limit_of_mine = (float)((double)clip * sqrt(about_mean / (double)D));
        for_each_bucket<NB>([&](auto q) {
            constexpr int kQ = decltype(q)::value;
            const float limit = readlane_f32(limit_of_mine, (int)reverse6(kQ));
#pragma unroll
            for (int j = 0; j < E; ++j) v[kQ * E + j] = clipped(v[kQ * E + j], limit);
        });
    }
    // From here on lane l works for bucket q(l); the lane with the free bits clear ("home") and the one
    // above it divide the lower and the upper side of that bucket.
    const double total = reduce_buckets<NB, double>(
        lane,
        [&](auto q) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const float x = v[decltype(q)::value * E + j];
                s += (double)(SIGN ? fabsf(x) : x);
            }
            return s;
        },
        add);
    const float trust_above = 1e-3f * reduce_buckets<NB, float>(  // see bingrad_bucket
                                          lane,
                                          [&](auto q) {
                                              float m = 0.0f;
#pragma unroll
                                              for (int j = 0; j < E; ++j) m = fmaxf(m, fabsf(v[decltype(q)::value * E + j]));
                                              return m;
                                          },
                                          larger);
    float b0 = (float)(total / (double)D);
    const bool upper = (lane & 1u) != 0;
    const bool home = (lane & kFreeBits) == 0;

    double b_lo = 0.0, b_hi = 0.0;
    uint32_t word_lo = 0, word_hi = 0;  // lane j ends up holding packed word j of the chunk
    uint32_t prev_n_lo = 0xFFFFFFFFu;
    if constexpr (SIGN) {  // Scaled SignSGD: see bingrad_bucket
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const uint64_t hi_mask = ~__ballot(v[j] < 0.0f);
            word_lo = writelane(word_lo, (uint32_t)hi_mask, j);
            word_hi = writelane(word_hi, (uint32_t)(hi_mask >> 32), j);
        }
        b_hi = total / (double)D;
        b_lo = -b_hi;
    } else
    for (uint32_t it = 0;; ++it) {
        uint32_t n_lo = 0;
        const double s_lo = reduce_buckets<NB, double>(
            lane,
            [&](auto q) {
                constexpr int kQ = decltype(q)::value;
                const float threshold = readlane_f32(b0, (int)reverse6(kQ));
                double s = 0.0;
                uint32_t below = 0;
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    const int reg = kQ * E + j;
                    const bool lo = v[reg] < threshold;
                    const uint64_t lo_mask = __ballot(lo);
                    const uint64_t hi_mask = ~lo_mask;
                    below += (uint32_t)__popcll(lo_mask);
                    s += (double)(lo ? v[reg] : 0.0f);
                    word_lo = writelane(word_lo, (uint32_t)hi_mask, reg);
                    word_hi = writelane(word_hi, (uint32_t)(hi_mask >> 32), reg);
                }
                n_lo = writelane(n_lo, below, (int)reverse6(kQ));
                return s;
            },
            add);
        n_lo = dpp_u32<kDppXor1From0>(n_lo);
        double s_hi = total - s_lo;
        const bool doubtful = !(fabs(s_hi) >= (double)trust_above);
        if (__ballot(doubtful) != 0) {
            const double direct = reduce_buckets<NB, double>(
                lane,
                [&](auto q) {
                    constexpr int kQ = decltype(q)::value;
                    const float threshold = readlane_f32(b0, (int)reverse6(kQ));
                    double s = 0.0;
#pragma unroll
                    for (int j = 0; j < E; ++j) s += (double)(!(v[kQ * E + j] < threshold) ? v[kQ * E + j] : 0.0f);
                    return s;
                },
                add);
            if (doubtful) s_hi = direct;
        }
        const uint32_t n_hi = D - n_lo;
        const double num = upper ? s_hi : s_lo;
        const uint32_t den = upper ? n_hi : n_lo;
        const double quot = num / (double)(den > 0 ? den : 1u);
        const double other = dpp_f64<kDppXor1>(quot);
        const double mean_lo = upper ? other : quot, mean_hi = upper ? quot : other;
        b_lo = n_lo > 0 ? mean_lo : mean_hi;  // constant bucket: both levels equal
        b_hi = n_hi > 0 ? mean_hi : mean_lo;
        // Further threshold updates are identities for a bucket once its partition repeats.
        if (it == iters || __ballot(home && n_lo != prev_n_lo) == 0) break;
        prev_n_lo = n_lo;
        b0 = (float)((b_lo + b_hi) * 0.5);
    }

    const uint32_t q = (__brev(lane) >> 26) & (uint32_t)(tree_of(NB) - 1);
    if (home && q < (uint32_t)NB) {
        float2 pair;
        pair.x = (float)b_lo;
        pair.y = (float)b_hi;
        *reinterpret_cast<float2*>(levels + ((size_t)chunk * NB + q) * 2) = pair;
    }
    if (lane < (uint32_t)R) codes[(size_t)chunk * R + lane] = ((uint64_t)word_hi << 32) | word_lo;
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------
template <int E>
void launch_bingrad(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes,
                    hipStream_t st)
{
    const dim3 grid((nb + kBinGradWaves - 1) / kBinGradWaves), block(kWave * kBinGradWaves);
    const bool clip = p->clip_factor > 0.0f, sign = p->scheme == OGQ_SCALED_SIGN;
#define OGQ_LAUNCH(CLIP, SIGN)                                                                                        \
    launch_kernel((bingrad_quantize_kernel<E, CLIP, SIGN>), grid, block, st, g, n, p->bucket_size,           \
                       p->level_iters, p->clip_factor, nb, lv, static_cast<uint64_t*>(codes))
    if (sign) {
        if (clip) OGQ_LAUNCH(true, true);
        else OGQ_LAUNCH(false, true);
    } else {
        if (clip) OGQ_LAUNCH(true, false);
        else OGQ_LAUNCH(false, false);
    }
#undef OGQ_LAUNCH
}

template <int W, int E = 32>
void launch_bingrad_team(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes,
                         hipStream_t st)
{
    const dim3 grid(nb), block(W * kWave);
    const bool clip = p->clip_factor > 0.0f, sign = p->scheme == OGQ_SCALED_SIGN;
#define OGQ_LAUNCH(CLIP, SIGN)                                                                               \
    launch_kernel((bingrad_team_kernel<W, E, CLIP, SIGN>), grid, block, st, g, n, p->bucket_size,   \
                       p->level_iters, p->clip_factor, nb, lv, static_cast<uint64_t*>(codes))
    if constexpr (E <= 32) {  // 64 registers of data leave no room for the clipping passes: the caller picks E = 32
        if (clip) {
            if (sign) OGQ_LAUNCH(true, true);
            else OGQ_LAUNCH(true, false);
            return;
        }
    }
    if constexpr (W < 16) {  // (without clipping the caller never asks for 16 wavefronts: see launch_two_level)
        if (sign) OGQ_LAUNCH(false, true);
        else OGQ_LAUNCH(false, false);
    } else {
        launch_status() = hipErrorInvalidDeviceFunction;
    }
#undef OGQ_LAUNCH
}

template <int E>
void launch_bingrad_chunks(const float* g, size_t n, const ogq_params_t* p, float* lv, void* codes, hipStream_t st)
{
    constexpr uint32_t CHUNK = 64u * E * buckets_of_a_wavefront(E);
    const uint32_t chunks = (uint32_t)(n / CHUNK), rest = (uint32_t)(n % CHUNK);
    const uint32_t waves = chunks + (rest + p->bucket_size - 1) / p->bucket_size;
    const dim3 grid((waves + kBinGradWaves - 1) / kBinGradWaves), block(kWave * kBinGradWaves);
    const bool clip = p->clip_factor > 0.0f, sign = p->scheme == OGQ_SCALED_SIGN;
#define OGQ_LAUNCH(CLIP, SIGN)                                                                                        \
    launch_kernel((bingrad_chunk_kernel<E, CLIP, SIGN>), grid, block, st, g, chunks, rest, p->level_iters, p->clip_factor, lv, \
                  static_cast<uint64_t*>(codes))
    if (sign) {
        if (clip) OGQ_LAUNCH(true, true);
        else OGQ_LAUNCH(false, true);
    } else {
        if (clip) OGQ_LAUNCH(true, false);
        else OGQ_LAUNCH(false, false);
    }
#undef OGQ_LAUNCH
}

// Number of buckets from which several of them share a wavefront.  Below, every SIMD has a wavefront or two anyway and one with more
// buckets only takes longer; threshold updates add to that.  profiles/bingrad_scan.txt has both sides for every size, tests/test_dispatch.py
// holds the limits against it.  us, one bucket per wavefront -> several, of BinGrad-b, its two updates, Scaled SignSGD:
//   64    8192 buckets 4.4 -> 4.2, 6.3 -> 6.8, 3.3 -> 2.9; 10240: 4.6 -> 4.2, 7.2 -> 6.8, 3.3 -> 2.9; clipped, 10240: 5.7 -> 6.1, 8.4 -> 8.3, 4.1 -> 4.8;
//         12288: 6.4 -> 6.1, 9.6 -> 8.3, 4.6 -> 4.8
//   128   4608: 3.4 -> 3.6, 4.9 -> 5.8, 2.7 -> 2.8; 6656: 3.9 -> 3.6, 5.8 -> 5.8, 2.9 -> 2.8; clipped, 12288: 6.8 -> 5.9, 9.9 -> 8.5, 4.7 -> 4.4
//   256   4608: 3.8 -> 3.8, 5.4 -> 6.2, 3.0 -> 2.9; 6656: 4.3 -> 4.1, 6.4 -> 6.4, 3.3 -> 3.2; clipped, 7680: 5.6 -> 5.1, 8.1 -> 7.4, 4.1 -> 3.9
//   512   6144: 4.3 -> 4.4, 6.7 -> 6.7, 3.1 -> 3.4; 6656: 4.6 -> 4.5, 7.3 -> 6.8, 3.3 -> 3.5; clipped 5.8 -> 5.5, 8.8 -> 7.8, 4.3 -> 4.4
//   1024  4096: 4.7 -> 4.7, 7.0 -> 7.3, 3.7 -> 3.7; 4608: 5.3 -> 5.2, 8.1 -> 8.2, 4.5 -> 3.9; 5632: 5.8 -> 5.9, 9.0 -> 9.5, 4.9 -> 4.4; 6656: 6.7 -> 6.1, 10.1 -> 9.8,
//         5.4 -> 4.8; clipped 7.9 -> 8.0, 11.6 -> 11.6, 6.3 -> 6.1
// A size between two of these leaves registers of the one-bucket kernel empty, and shares earlier:
//   192   4096: 3.7 -> 3.5, 5.0 -> 5.4, 2.9 -> 2.8; 4608: 4.1 -> 3.5, 5.8 -> 5.4, 3.2 -> 2.8; clipped, 6656: 6.0 -> 5.5, 8.4 -> 8.0, 4.7 -> 4.3
//   704   512: 3.2 -> 3.1, 4.3 -> 4.5, 2.7 -> 2.5; 768: 3.6 -> 3.1, 5.1 -> 4.5, 2.9 -> 2.5; clipped 4.2 -> 3.6, 5.8 -> 5.0, 3.6 -> 3.0
static uint32_t several_buckets_from(uint32_t d, bool clipped, bool updates)
{
    switch (d) {
        case 64: return updates ? 10240u : clipped ? 12288u : 8192u;
        case 128: return clipped ? 12288u : updates ? 6656u : 4608u;
        case 192: return clipped ? 6656u : 4608u;
        case 256: return clipped ? 7680u : updates ? 6656u : 4608u;
        case 512: return 6656u;
        case 1024: return clipped || updates ? 6656u : 4608u;
        case 704: case 768: return 768u;
        default: return d < 512u ? 4608u : 2560u;
    }
}

void launch_two_level(const float* g, size_t n, const ogq_params_t* p, float* lv, void* codes, hipStream_t st)
{
    const uint32_t d = p->bucket_size;
    const uint32_t nb = (uint32_t)(n / d + (n % d != 0));
    const uint32_t regs = d / 64;
    // Buckets of up to 1024 elements: several per wavefront where there are enough of them (what is left, fewer than 2048 elements, gets
    // one wavefront per bucket in the same launch: one of its own cost 2.8 us).
    const bool updates = p->scheme == OGQ_BINGRAD_B && p->level_iters > 0u;
    if (regs <= 16 && nb >= several_buckets_from(d, p->clip_factor > 0.0f, updates)) {
        switch (regs) {
#define OGQ_CASE(E) case E: launch_bingrad_chunks<E>(g, n, p, lv, codes, st); return
            OGQ_CASE(1); OGQ_CASE(2); OGQ_CASE(3); OGQ_CASE(4); OGQ_CASE(5); OGQ_CASE(6); OGQ_CASE(7); OGQ_CASE(8);
            OGQ_CASE(9); OGQ_CASE(10); OGQ_CASE(11); OGQ_CASE(12); OGQ_CASE(13); OGQ_CASE(14); OGQ_CASE(15); OGQ_CASE(16);
#undef OGQ_CASE
        }
    }
    if (regs <= 1) launch_bingrad<1>(g, n, p, nb, lv, codes, st);
    else if (regs <= 2) launch_bingrad<2>(g, n, p, nb, lv, codes, st);
    else if (regs <= 4) launch_bingrad<4>(g, n, p, nb, lv, codes, st);
    else if (regs <= 8) launch_bingrad<8>(g, n, p, nb, lv, codes, st);
    else if (regs <= 16) launch_bingrad<16>(g, n, p, nb, lv, codes, st);
    else if (regs <= 32) {
        // A kernel for each size: no register without an element, no test whether there is one (25.6 M values in buckets of 1344 with
        // 32 registers -> 21: 22.2 -> 19.0 us, with clipping 38.7 -> 22.1).
        switch (regs) {
#define OGQ_CASE(E) case E: launch_bingrad<E>(g, n, p, nb, lv, codes, st); return
            OGQ_CASE(17); OGQ_CASE(18); OGQ_CASE(19); OGQ_CASE(20); OGQ_CASE(21); OGQ_CASE(22); OGQ_CASE(23); OGQ_CASE(24);
            OGQ_CASE(25); OGQ_CASE(26); OGQ_CASE(27); OGQ_CASE(28); OGQ_CASE(29); OGQ_CASE(30); OGQ_CASE(31); OGQ_CASE(32);
#undef OGQ_CASE
        }
    }
    else if (regs <= 64) launch_bingrad_team<2>(g, n, p, nb, lv, codes, st);
    else if (regs <= 128) launch_bingrad_team<4>(g, n, p, nb, lv, codes, st);
    else if (p->clip_factor > 0.0f) {
        // the clipping passes need the registers a second 2048 elements per wavefront would take
        if (regs <= 256) launch_bingrad_team<8>(g, n, p, nb, lv, codes, st);
        else launch_bingrad_team<16>(g, n, p, nb, lv, codes, st);
    } else if (regs <= 256 && (nb <= 512 || (regs == 256 && (p->level_iters == 0 || p->scheme == OGQ_SCALED_SIGN)))) {
        // Twice the wavefronts per bucket: faster while there are at most two buckets per CU (up to 8 %), and at any number
        // (2 to 10 %) where every register holds an element and one pass over the bucket is all there is.
        launch_bingrad_team<8>(g, n, p, nb, lv, codes, st);
    } else if (regs <= 256) launch_bingrad_team<4, 64>(g, n, p, nb, lv, codes, st);
    else launch_bingrad_team<8, 64>(g, n, p, nb, lv, codes, st);
}

}  // namespace ogq
