// Internal header of libogq: the random-rounding quantize kernels for small buckets of long gradients, four or eight buckets per
// wavefront.  Included by rounding_part.hip after rounding_kernels.h, whose encoder it uses.  Compile with -ffp-contract=off.
#ifndef OGQ_ROW_KERNELS_H
#define OGQ_ROW_KERNELS_H

#include "group_solve.h"

namespace ogq {

// ----------------------------------------------------------------------------------------------
// ORQ, Linear-s and evenly spaced levels for bucket sizes d = 64 m up to 512, 64 / LANES whole buckets per wavefront: row r of LANES =
// 16 or 8 lanes owns bucket r of the wavefront's span and holds its elements 4 LANES c + 4i + {0..3} in lane i, chunk c.
//
// What bounds it: vector-instruction issue.  With one bucket per wavefront (orq_quantize_kernel) a bucket of 512 elements costs 1,400
// instructions at nine levels, of which its 8 x 64 elements need about 350: the solves, reductions and scans are the same for
// 2048 elements as for 512, and in a solve all 64 lanes do one bucket's arithmetic.  Here every such instruction works for four or
// eight buckets.  From five levels on a row of 16 lanes is two groups of 8, one for each chain of solves (group_solve.h): 4 steps
// instead of 7 at nine levels.  Buckets of 128 take rows of 8 lanes: what a wavefront does once it does for eight of them.
// 25.6 M values, one bucket per wavefront -> four, serial solves -> now: nine levels, buckets of 512, clipping 129 -> 78.6 -> 62.5 us; three
// levels, buckets of 128 69 -> 43.7 -> 38.7; eight levels, two sweeps, 512: 137.6 -> 93.4 (the last two).
// The phases are those of orq_bucket: extremes, grouping in LDS by value bins (ScaledBins), fp64 prefix, level solves, encode.
//
// Positions and bin counts are kept in bytes (times 4), bin starts as offsets into the wavefront's values; what a bin's counter hands an element
// leaves the scatter two vector instructions (counter_start).  Buckets of 256 in rows of 8 lanes were slower (1 to 27 %: half the wavefronts, twice the registers).
// ----------------------------------------------------------------------------------------------
// LDS of a wavefront.  At 512 elements per bucket it decides how many wavefronts a CU holds (14 with 11.5 KB), so the bin counts lie
// where the values are grouped afterwards, and bin starts take 16 bits.
template <int LANES, int C, int S>
struct alignas(16) RowLds {
    static constexpr int ROWS = 64 / LANES;
    static constexpr int D = 4 * LANES * C;  // element capacity of a row
    // Bins.  Eight rows of three levels: 80, so that 25 wavefronts of 6240 bytes fit a CU's LDS (128 bins: 21), and a lane's ten counters are read
    // without bank conflicts; with counter_start and the sum of compares, 25.6 M values in buckets of 128 38.4 -> 34.4 us on one card, 38.6 -> 37.5 on
    // another.
    static constexpr int B = LANES == 8 && S <= 3 ? 80 : 128, HALF = B / 2;
    static constexpr int CHAINS = S > 4 && LANES == 16 ? 2 : 1;  // groups of lanes that solve a bucket's levels
    static constexpr int GROUP = LANES / CHAINS;
    static constexpr int BLOCK = D >= 512 || GROUP > 8 ? 16 : 8;  // positions per entry of the fp64 prefix
    static constexpr bool SUMS = S > 3;  // (with one interior level the solve reads the bucket's total alone)
    static constexpr bool END_OF_BUCKET = true, LEAF = false;  // (group_solve)
    union {
        uint32_t bin_count[ROWS * B];  // bytes: 4 per element
        uint32_t grouped[ROWS * D];    // fp32 bit patterns by bin, row after row
    };
    uint16_t bin_start[ROWS * B + 2];  // byte offset of each bin's first position in `grouped`
    double prefix[SUMS ? ROWS * (D / BLOCK) : 1];
    GroupLevel level[ROWS][S];
    unsigned long long exact_limb[kExactLimbs];
};

// Inclusive scans over the lanes of every row.
template <int LANES>
__device__ __forceinline__ uint32_t row_scan_u32(uint32_t x, uint32_t i)
{
    if constexpr (LANES == 16) {
        x += dpp_or_zero_u32<kDppRowShr1, 0xF>(x);
        x += dpp_or_zero_u32<kDppRowShr2, 0xF>(x);
        x += dpp_or_zero_u32<kDppRowShr4, 0xF>(x);
        x += dpp_or_zero_u32<kDppRowShr8, 0xF>(x);
    } else {
        // (the shifts reach into the other half of 16 lanes)
        uint32_t y = dpp_or_zero_u32<kDppRowShr1, 0xF>(x);
        x += i >= 1u ? y : 0u;
        y = dpp_or_zero_u32<kDppRowShr2, 0xF>(x);
        x += i >= 2u ? y : 0u;
        y = dpp_or_zero_u32<kDppRowShr4, 0xF>(x);
        x += i >= 4u ? y : 0u;
    }
    return x;
}

template <int LANES>
__device__ __forceinline__ double row_scan_f64(double x, uint32_t i)
{
    if constexpr (LANES == 16) return row_inclusive_scan_f64<16>(x);
    double y = dpp_or_zero_f64<kDppRowShr1, 0xF>(x);
    x += i >= 1u ? y : 0.0;
    y = dpp_or_zero_f64<kDppRowShr2, 0xF>(x);
    x += i >= 2u ? y : 0.0;
    y = dpp_or_zero_f64<kDppRowShr4, 0xF>(x);
    x += i >= 4u ? y : 0.0;
    return x;
}

template <int LANES>
__device__ __forceinline__ float row_sum_f32(float x)
{
    x += dpp_f32<kDppXor1>(x);
    x += dpp_f32<kDppXor2>(x);
    x += dpp_f32<kDppHalfMirror>(x);
    if constexpr (LANES == 16) x += dpp_f32<kDppMirror>(x);
    return x;
}

// The reload function of the encoder: g = the row's first element, limit = its clipping threshold (infinity: none).
template <int LANES>
struct ReloadRow {
    const float* g;
    float limit;
    __device__ __forceinline__ void operator()(uint32_t c, float (&y)[4]) const
    {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            y[k] = clipped(g[4u * LANES * c + 4u * (threadIdx.x & (uint32_t)(LANES - 1)) + (uint32_t)k], limit);
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

// The whole buckets of `chunks` * 4 LANES elements that begin at global element `begin`; bucket = the first one's index.
template <int LANES, int C, int S, int BITS, bool EXACT, int RULE>
__device__ __forceinline__ void orq_rows_span(RowLds<LANES, C, S>& lds, const float* __restrict__ grad, uint32_t chunks, size_t begin,
                                              uint32_t bucket, uint32_t sweeps, float clip, uint64_t seed, uint64_t index_offset,
                                              float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    static_assert(RULE == kOptimal || RULE == kEven || RULE == kLinear, "rules of this kernel");
    using Lds = RowLds<LANES, C, S>;
    constexpr uint32_t B = Lds::B, HALF = B / 2, D = Lds::D;
    constexpr uint32_t PER = B / LANES;  // bins per lane
    constexpr uint32_t PIECE = PER % 4u == 0u ? 4u : 2u;  // counters read or written at once
    struct alignas(4 * PIECE) CounterPiece {
        uint32_t at[PIECE];
    };
    constexpr bool GROUPED = S > 2 && RULE != kEven;
    constexpr bool SUMS = RULE == kOptimal && Lds::SUMS;
    const uint32_t lane = threadIdx.x & 63u, row = lane / LANES, i = lane & (uint32_t)(LANES - 1);
    const uint32_t len = 4u * LANES * chunks;
    const float* g = grad + begin + row * len;

    float v[C][4];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[c][k] = 0.0f;
    for_row_chunks<C, EXACT>(chunks, [&](int c) {
        const floatx4 q = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(g + 4 * LANES * c + 4 * i));
        v[c][0] = q.x; v[c][1] = q.y; v[c][2] = q.z; v[c][3] = q.w;
    });
    const uint32_t grouped_at = (uint32_t)(uintptr_t)((LdsWord*)lds.grouped);
    if constexpr (GROUPED) {
        const uint32_t count = counter_start((uint32_t)(uintptr_t)((LdsHalf*)lds.bin_start), grouped_at, PIECE * lane);
#pragma unroll
        for (uint32_t q = 0; q < PER / PIECE; ++q) {  // (neighbours write neighbouring counters: no bank conflicts)
            CounterPiece x;
#pragma unroll
            for (uint32_t t = 0; t < PIECE; ++t) x.at[t] = count + ((64u * PIECE * q + t) << 17);
            reinterpret_cast<CounterPiece*>(lds.bin_count)[64u * q + lane] = x;
        }
    }
    float limit = __uint_as_float(0x7F800000u);  // clipping threshold
    if (clip > 0.0f) {  // the same for every thread of the grid
        float(&flat)[4 * C] = reinterpret_cast<float(&)[4 * C]>(v);
        limit = clip_in_registers<4 * C>(
            flat, len, clip, [&](int j) { return EXACT || (uint32_t)(j >> 2) < chunks; },
            [&](double& x, double& y) {
                x = row_sum_f64<LANES>(x, lane);
                y = row_sum_f64<LANES>(y, lane);
            });
    }

    // ---- extremes of every row ---------------------------------------------------------------------
    float low = v[0][0], high = v[0][0], sample = 0.0f;
    for_row_chunks<C, EXACT>(chunks, [&](int c) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            low = fminf(low, v[c][k]);
            high = fmaxf(high, v[c][k]);
        }
        if constexpr (GROUPED) sample += __builtin_fabsf(v[c][0]);
    });
    low = key_to_float(row_min_u32<LANES>(float_to_key(low + 0.0f), lane));  // (-0 -> +0)
    high = key_to_float(row_max_u32<LANES>(float_to_key(high + 0.0f), lane));
    const uint32_t mag_max = umax32(__float_as_uint(low) & 0x7FFFFFFFu, __float_as_uint(high) & 0x7FFFFFFFu);

    if constexpr (GROUPED) {
        // mean magnitude of every fourth element
        const float mean = row_sum_f32<LANES>(sample) * __builtin_amdgcn_rcpf((float)(uint32_t)(LANES * (EXACT ? (uint32_t)C : chunks)));
        const ScaledBins bins = scaled_bins<(int)HALF>(mean, mag_max);

        // ---- histogram: the returning LDS add hands every element its position inside its bin --------
        uint32_t slot[C][4];  // what the bin's counter returned (counter_start)
        {
            wave_lds_sync();
            const float zero = opaque_zero();
            const uint64_t origin = bin_origin(bins);
            const uint32_t middle = (uint32_t)(uintptr_t)((LdsWord*)lds.bin_count) + 4u * (B * row + HALF);
            for_row_chunks<C, EXACT>(chunks, [&](int c) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const uint32_t counter = middle + 4u * (uint32_t)signed_bin<(int)HALF>(v[c][k] + zero, bins, origin);
                    slot[c][k] = __hip_atomic_fetch_add((LdsWord*)(uintptr_t)counter, 4u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            });
            wave_lds_sync();
        }

        // ---- bin starts: exclusive prefix over the row's counts (lane i owns PER bins) ----------------
        {
            const CounterPiece* mine = reinterpret_cast<const CounterPiece*>(lds.bin_count) + PER / PIECE * lane;
            uint32_t count[PER], total = 0;
#pragma unroll
            for (uint32_t q = 0; q < PER / PIECE; ++q) {
                const CounterPiece x = mine[q];
#pragma unroll
                for (uint32_t t = 0; t < PIECE; ++t) count[PIECE * q + t] = x.at[t];
            }
#pragma unroll
            for (uint32_t t = 0; t < PER; ++t) total += count[t];
            // (the lower 16 bits are what counts)
            total -= PER * grouped_at;
            uint32_t start = 4u * D * row + row_scan_u32<LANES>(total, i) - total;
            uint32_t* pairs = reinterpret_cast<uint32_t*>(lds.bin_start) + PER / 2u * lane;
#pragma unroll
            for (uint32_t t = 0; t < PER / 2u; ++t) {
                const uint32_t next = start + count[2 * t] - grouped_at;
                pairs[t] = two_starts(start, next);
                start = next + count[2 * t + 1] - grouped_at;
            }
            if (lane == 63u) lds.bin_start[Lds::ROWS * B] = (uint16_t)start;
        }
        wave_lds_sync();  // (all counts are read before values take their place)

        // ---- scatter the values into their bins (bin starts of a group of chunks read before its writes) ----
        char* grouped = reinterpret_cast<char*>(lds.grouped);
        {
            constexpr int BATCH = C < 4 ? C : 4;
#pragma unroll
            for (int c0 = 0; c0 < C; c0 += BATCH) {
#pragma unroll
                for (int c = c0; c < c0 + BATCH; ++c)
                    if (EXACT || (uint32_t)c < chunks) {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            slot[c][k] = place_in_bin(slot[c][k]);
                    }
#pragma unroll
                for (int c = c0; c < c0 + BATCH; ++c)
                    if (EXACT || (uint32_t)c < chunks) {
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            *(LdsWord*)(uintptr_t)slot[c][k] = __float_as_uint(v[c][k]);
                    }
            }
            wave_lds_sync();
        }

        // ---- fp64 prefix of the grouped values, one entry per BLOCK positions (lane i: 4 C positions) ------
        double total = 0.0, bound = 0.0;
        if constexpr (SUMS) {
            constexpr uint32_t MINE = 4u * C, BLOCK = Lds::BLOCK;
            constexpr uint32_t PIECES = (MINE < BLOCK ? MINE : BLOCK) / 4u;  // 16-byte pieces of an entry that are this lane's
            const float4* from = reinterpret_cast<const float4*>(lds.grouped + row * D + MINE * i);
            double part = 0.0, before[MINE / BLOCK > 0 ? MINE / BLOCK : 1];
#pragma unroll
            for (uint32_t e = 0; e < (uint32_t)C / PIECES; ++e) {
                before[e] = part;
#pragma unroll
                for (uint32_t q = 0; q < PIECES; ++q) {
                    // every lane begins at another piece, so that the lanes meet different LDS banks
                    const uint32_t at = e * PIECES + ((q + i) & (PIECES - 1u));
                    const bool exists = EXACT || MINE * i + 4u * at < len;
                    const float4 x = from[at];
                    part += (double)(exists ? x.x : 0.0f);
                    part += (double)(exists ? x.y : 0.0f);
                    part += (double)(exists ? x.z : 0.0f);
                    part += (double)(exists ? x.w : 0.0f);
                }
            }
            const double incl = row_scan_f64<LANES>(part, i);
            if constexpr (MINE >= BLOCK) {
                double* entry = lds.prefix + row * (D / BLOCK) + MINE / BLOCK * i;
#pragma unroll
                for (uint32_t e = 0; e < MINE / BLOCK; ++e) entry[e] = (incl - part) + before[e];
            } else {
                // (two lanes share an entry)
                if (i % (BLOCK / MINE) == 0u) lds.prefix[row * (D / BLOCK) + i / (BLOCK / MINE)] = incl - part;
            }
            total = lane_fetch_f64(incl, lane | (uint32_t)(LANES - 1));
        } else if constexpr (RULE == kOptimal) {
            double part = 0.0;
            for_row_chunks<C, EXACT>(chunks, [&](int c) {
#pragma unroll
                for (int k = 0; k < 4; ++k) part += (double)v[c][k];
            });
            total = row_sum_f64<LANES>(part, lane);
        }

        if constexpr (RULE == kOptimal) {
            // ---- may the fp64 sums round?  (small elements sit in the bins next to zero: see any_tiny_element) ----
            constexpr uint32_t SAFE = safe_binades(D);
            const uint32_t biased = mag_max >> 23;
            uint32_t tiny = 0u;
            if (biased > SAFE) {
                const uint32_t mag_safe = (biased - SAFE) << 23;
                const uint32_t near = magnitude_bin<(int)HALF>(__uint_as_float(mag_safe), bins) + 1u;
                const uint16_t* middle = lds.bin_start + row * B + HALF;
                const uint32_t last = umin32(middle[near], 4u * (row * D + len));
                for (uint32_t p = middle[-(int)near] + 4u * i; p < last; p += 4u * LANES) {
                    const uint32_t magnitude = *reinterpret_cast<const uint32_t*>(grouped + p) & 0x7FFFFFFFu;
                    if (magnitude != 0u && magnitude < mag_safe) tiny = 1u;
                }
            }
            bound = row_max_u32<LANES>(tiny, lane) != 0u ? sum_error_bound_of(mag_max, D) : 0.0;
        }
        // ---- level records of the ends (lane i: those of the levels i, i + LANES, ...) ---------------------
#pragma unroll
        for (uint32_t k = i; k < (uint32_t)S; k += LANES) {
            const bool top = k == (uint32_t)(S - 1);
            GroupLevel end;
            end.value = top ? high : low;
            end.count_lt = end.count_le = (uint16_t)(top ? len : 0u);
            end.sum_lt = end.sum_le = top ? total : 0.0;
            end.rank = 0u;
            lds.level[row][k] = end;
        }
        wave_lds_sync();

        // ---- the levels ------------------------------------------------------------------------------------
        const GroupBucket view{grouped, lds.bin_start + row * B + HALF, lds.prefix, lds.level[row], lds.exact_limb, bins, row * D, len, bound};
        if constexpr (RULE == kLinear) {
            GroupTie tie{0.0f, 0u};
#pragma unroll 1
            for (uint32_t k = 1; k + 1 < (uint32_t)S; ++k) {
                const float value = group_element<LANES, Lds>(view, k * (len - 1u) / (uint32_t)(S - 1), tie, lane);
                if (i == 0u) lds.level[row][k].value = value;
            }
            wave_lds_sync();
        } else {
            group_solve_levels<Lds::GROUP, Lds::CHAINS, S, Lds>(view, sweeps, lane);
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
    if constexpr (S > LANES) {
        if (i == 0u) levels[(size_t)(bucket + row) * S + (S - 1)] = lv[S - 1];
    }

    const EncodeRange range{256u * chunks, (index_offset + begin) >> 2, row * (len / 4u) + i, len / 64u, (uint32_t)seed,
                            (uint32_t)(seed >> 32), codes32 + begin / 64 * (2 * BITS)};
    constexpr Fill FILL = EXACT ? Fill::kAll : Fill::kWholeChunks;
    if constexpr (GROUPED && S > kScaledWidthLevels)  // (72 bytes from table to table: other LDS banks)
        encode_all<Rows<LANES>, C, S, BITS, FILL>(v, lv, range, ReloadRow<LANES>{g, limit},
                                                  PairsInLds{(uint32_t)(uintptr_t)((LdsWord*)lds.grouped) + 72u * row, i == 0u});
    else
        encode_all<Rows<LANES>, C, S, BITS, FILL, RULE == kEven && S == 3>(v, lv, range, ReloadRow<LANES>{g, limit});
}

// (Eight rows of three levels: 80 registers, six wavefronts per SIMD, which their LDS allows.)
// Blocks 0 .. singles - 1 take the buckets behind the last whole span (a few whole ones and a cut-off one), one each as in
// orq_quantize_kernel and first so that they do not end the launch alone; the others take a span each.
template <int LANES, int C, int S, int BITS, bool EXACT, int RULE>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(C == 8 ? (EXACT ? 4 : 3) : LANES == 8 && S <= 3 ? 6 : 1))) void orq_rows_kernel(const float* __restrict__ grad, size_t n, uint32_t bucket_size,
                                                         uint32_t sweeps, float clip, uint32_t num_buckets, uint32_t spans,
                                                         uint64_t seed, uint64_t index_offset, float* __restrict__ levels,
                                                         uint32_t* __restrict__ codes32)
{
    using Span = RowLds<LANES, C, S>;
    constexpr int CB = Span::D <= 256 ? 1 : 2;  // chunks of 256 elements of a bucket
    using Single = OrqLds<OrqShape<CB>::D, OrqShape<CB>::B, S>;
    __shared__ __attribute__((aligned(16))) unsigned char raw[sizeof(Span) > sizeof(Single) ? sizeof(Span) : sizeof(Single)];
    const uint32_t singles = num_buckets - Span::ROWS * spans;
    if (blockIdx.x < singles) {
        const uint32_t bucket = Span::ROWS * spans + blockIdx.x;
        const size_t begin = (size_t)bucket * bucket_size;
        const size_t rest = n - begin;
        const uint32_t len = rest < bucket_size ? (uint32_t)rest : bucket_size;
        orq_bucket<CB, S, BITS, false, true, RULE>(*reinterpret_cast<Single*>(raw), grad + begin, len, begin, bucket, sweeps, clip,
                                                   seed, index_offset, levels, codes32);
    } else {
        const uint32_t bucket = Span::ROWS * (blockIdx.x - singles);
        orq_rows_span<LANES, C, S, BITS, EXACT, RULE>(*reinterpret_cast<Span*>(raw), grad, bucket_size / (4u * LANES),
                                                      (size_t)bucket * bucket_size, bucket, sweeps, clip, seed, index_offset, levels, codes32);
    }
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------
// Which rules and level counts the dispatch in rounding_part.hip gives to rows of LANES; the others are not compiled, and asking for one fails
// (see wave_serves).
template <int LANES, int C>
constexpr bool rows_serve(int S, int rule)
{
    return !(LANES == 16 && C == 2 && S >= 5 && rule == kLinear);  // (buckets of 128: rows of 8 lanes or sorted_small_kernel)
}

template <int LANES, int C, int S, int BITS, bool EXACT, int RULE>
void launch_rows(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if constexpr (rows_serve<LANES, C>(S, RULE)) {
        constexpr uint32_t ROWS = RowLds<LANES, C, S>::ROWS;
        const uint32_t spans = (uint32_t)(n / p->bucket_size / ROWS);
        launch_kernel((orq_rows_kernel<LANES, C, S, BITS, EXACT, RULE>), dim3(nb - ROWS * spans + spans), dim3(kWave), st, g, n, p->bucket_size,
                      p->level_iters, p->clip_factor, nb, spans, p->seed, p->index_offset, lv, static_cast<uint32_t*>(codes));
    } else {
        launch_status() = hipErrorInvalidDeviceFunction;
    }
}

template <int LANES, int C, bool EXACT>
bool launch_rows_levels(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    switch (p->scheme) {
        case OGQ_ORQ:
            switch (p->bits) {
                case 1: launch_rows<LANES, C, 2, 1, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
                case 2: launch_rows<LANES, C, 4, 2, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
                default: launch_rows<LANES, C, 8, 3, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
            }
        case OGQ_ORQ_PAPER:
            switch (p->bits) {
                case 2: launch_rows<LANES, C, 3, 2, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
                case 3: launch_rows<LANES, C, 5, 3, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
                default: launch_rows<LANES, C, 9, 4, EXACT, kOptimal>(g, n, p, nb, lv, codes, st); return true;
            }
        case OGQ_EVEN:
            switch (p->bits) {
                case 2: launch_rows<LANES, C, 3, 2, EXACT, kEven>(g, n, p, nb, lv, codes, st); return true;
                case 3: launch_rows<LANES, C, 5, 3, EXACT, kEven>(g, n, p, nb, lv, codes, st); return true;
                default: launch_rows<LANES, C, 9, 4, EXACT, kEven>(g, n, p, nb, lv, codes, st); return true;
            }
        case OGQ_LINEAR:
            switch (p->bits) {
                case 2: launch_rows<LANES, C, 3, 2, EXACT, kLinear>(g, n, p, nb, lv, codes, st); return true;
                case 3: launch_rows<LANES, C, 5, 3, EXACT, kLinear>(g, n, p, nb, lv, codes, st); return true;
                default: launch_rows<LANES, C, 9, 4, EXACT, kLinear>(g, n, p, nb, lv, codes, st); return true;
            }
        default: return false;  // BinGrad-pb
    }
}

}  // namespace ogq
#endif  // OGQ_ROW_KERNELS_H
