// Internal header of libogq: the quantize kernels of the schemes with random rounding (ORQ: Theorem 1, its
// discrete remark, Corollary 1, Algorithm 1 and the random rounding of Section 3.1 of arXiv 2002.11082;
// BinGrad-pb; evenly spaced and Linear-s levels) and their launcher templates.  Included by rounding_part.hip,
// which instantiates one bucket capacity per object file.  Compile with -ffp-contract=off: the rounding decision
// is specified operation by operation in fp32.
#ifndef OGQ_ROUNDING_KERNELS_H
#define OGQ_ROUNDING_KERNELS_H

#include <type_traits>

#include "device_common.h"
#include "launch.h"

namespace ogq {

// ----------------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): counter (c0, c1, 0, 0), key (k0, k1).
// ----------------------------------------------------------------------------------------------
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t k0, uint32_t k1, uint32_t (&r)[4])
{
    uint32_t c2 = 0, c3 = 0;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t pa = (uint64_t)0xD2511F53u * c0;
        const uint64_t pb = (uint64_t)0xCD9E8D57u * c2;
        // three-input exclusive or in one instruction (v_bitop3_b32, truth table 0x96)
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pb >> 32), c1, k0, 0x96);
        const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(pa >> 32), c3, k1, 0x96);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    r[0] = c0; r[1] = c1; r[2] = c2; r[3] = c3;
}

// The same where c1 is wave-uniform: the first two rounds are then partly scalar (one product and one exclusive or of
// each; written out because the compiler takes the scalar product for a vector one).  What depends on c1 and the key alone
// is made once and held in registers: the compiler would make it again behind every branch.  VECTOR: in vector registers.  An exclusive or with a
// scalar operand issues in four cycles, one of vector registers alone in little more than half of that where other wavefronts fill in, and a Philox
// block has 17 of them; but 19 moves and 19 registers come first.  They pay in the pool's draws, where they cost no wavefronts (143.7 M values in buckets of
// 4096, eight levels, 293 -> 287 us), and with three evenly spaced levels in whole buckets of 2048, which have few other instructions, although six wavefronts
// per SIMD are left of eight (scalar -> vector on two cards, 20 M values 16.2 -> 15.8, 17.2 -> 16.9; 25.6 M 19.9 -> 19.3, 21.4 -> 21.0; 50 M 36.9 -> 35.4, 37.8 -> 37.8).
// In buckets of 512, where it is five of seven, neither is the faster one (16.5 -> 16.3, 17.3 -> 17.1; 12 M 11.6 -> 12.0; 50 M 36.8 -> 35.9, 38.0 -> 38.3), with clipping nothing
// is left of it (24.3 -> 24.5), 8 wavefronts per bucket lose (25.6 M in buckets of 16384 23.9 -> 24.2), and so does ORQ-3 there (28.0 -> 29.4).
struct PhiloxWords {
    uint32_t first;       // k1
    uint32_t second[2];   // of round 2: what x0 and x2 are combined with
    uint32_t third;       // of round 3: what x2 is combined with
    uint32_t k0[8], k1[7];  // the keys of rounds 3 .. 10 and 4 .. 10
};

template <bool VECTOR>
__device__ __forceinline__ PhiloxWords philox_words(uint32_t c1, uint32_t k0, uint32_t k1)
{
    constexpr uint32_t kMulA = 0xD2511F53u, kWeylA = 0x9E3779B9u, kWeylB = 0xBB67AE85u;
    PhiloxWords w;
    const uint64_t qa = (uint64_t)kMulA * uniform_u32(c1 ^ k0);  // round 2, the product of the uniform word
    w.first = k1;
    w.second[0] = k0 + kWeylA;
    w.second[1] = (uint32_t)(qa >> 32) ^ (k1 + kWeylB);
    w.third = (uint32_t)qa ^ (k1 + 2u * kWeylB);
#pragma unroll
    for (uint32_t r = 0; r < 8; ++r) w.k0[r] = k0 + (r + 2u) * kWeylA;
#pragma unroll
    for (uint32_t r = 0; r < 7; ++r) w.k1[r] = k1 + (r + 3u) * kWeylB;
    auto hold = [](uint32_t& x) {
        if constexpr (VECTOR) {
            asm("" : "+v"(x));
        } else {
            x = uniform_u32(x);
            asm("" : "+s"(x));
        }
    };
    hold(w.first); hold(w.second[0]); hold(w.second[1]); hold(w.third);
#pragma unroll
    for (int r = 0; r < 8; ++r) hold(w.k0[r]);
#pragma unroll
    for (int r = 0; r < 7; ++r) hold(w.k1[r]);
    return w;
}

__device__ __forceinline__ void philox4x32_10_uniform_c1(uint32_t c0, const PhiloxWords& w, uint32_t (&r)[4])
{
    constexpr uint32_t kMulA = 0xD2511F53u, kMulB = 0xCD9E8D57u;
    const uint64_t pa = (uint64_t)kMulA * c0;                    // round 1: c2 = c3 = 0
    const uint64_t qb = (uint64_t)kMulB * ((uint32_t)(pa >> 32) ^ w.first);
    uint32_t x0 = (uint32_t)(qb >> 32) ^ w.second[0], x1 = (uint32_t)qb;
    uint32_t x2 = (uint32_t)pa ^ w.second[1], x3 = 0u;
#pragma unroll
    for (int round = 2; round < 10; ++round) {
        const uint64_t ra = (uint64_t)kMulA * x0, rb = (uint64_t)kMulB * x2;
        const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(rb >> 32), x1, w.k0[round - 2], 0x96);
        // (round 2: x3 and the key are both uniform)
        const uint32_t n2 = round == 2 ? (uint32_t)(ra >> 32) ^ w.third
                                       : __builtin_amdgcn_bitop3_b32((uint32_t)(ra >> 32), x3, w.k1[round > 2 ? round - 3 : 0], 0x96);
        x1 = (uint32_t)rb;
        x3 = (uint32_t)ra;
        x0 = n0;
        x2 = n2;
    }
    r[0] = x0; r[1] = x1; r[2] = x2; r[3] = x3;
}

// ----------------------------------------------------------------------------------------------
// ORQ quantize.  One wavefront (= one workgroup) owns one bucket.  Lane l holds, for chunk c, the
// four consecutive bucket elements 256*c + 4*l + {0,1,2,3} (one 16-byte load), which are also the
// four elements that share one Philox block.
//
// A level solve needs (a) counts and sums of the elements below a level and (b) the element of a
// given rank.  The bucket is therefore grouped once, in LDS, by a monotone bin of the value (sign,
// exponent and top mantissa bits, relative to the largest magnitude of the bucket; everything more
// than 16 binades below that shares the two centre bins).  The bin counts and the fp64 sums of blocks
// of positions are prefix-summed; after that a solve touches one bin: the element of the wanted rank is
// selected among the bin's keys, one per lane (select_rank), and the counts and sums below it are added
// to what lies before the bin.
//
// What bounds it: vector-instruction issue and, in the solves, a scalar chain.  A bucket of 2048 at four levels takes 1,918 vector
// and 771 scalar instructions, of which the solves about 500 each, in a chain of lane read, compare and scalar count;
// SQ_ACTIVE_INST_VALU / SQ_BUSY_CU_CYCLES is 0.85 (profiles/orq_cfg3_issue_counters_pmc.txt; 25.6 M values 51 us among other passes,
// 57 alone).
// ----------------------------------------------------------------------------------------------
// Order-preserving map of fp32 onto unsigned integers.
__device__ __forceinline__ uint32_t float_to_key(float f)
{
    const uint32_t u = __float_as_uint(f);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

__device__ __forceinline__ float key_to_float(uint32_t k)
{
    const uint32_t u = (k & 0x80000000u) ? (k ^ 0x80000000u) : ~k;
    return __uint_as_float(u);
}

// Order of the greedy solves (Algorithm 1): the level in the middle of [l, r] is solved from the
// two outer levels, then both halves are treated the same way; the middle index is rounded down
// when s is not of the form 2^K + 1.  Each step is packed as 4 bits of k, l, r; five steps per word.
struct GreedyOrder {
    uint64_t packed[2];
    int count;
};

constexpr void greedy_visit(GreedyOrder& o, int l, int r)
{
    if (r - l < 2) return;
    const int mid = (l + r) / 2;
    o.packed[o.count / 5] |= (uint64_t)(mid | (l << 4) | (r << 8)) << (12 * (o.count % 5));
    ++o.count;
    greedy_visit(o, l, mid);
    greedy_visit(o, mid, r);
}

template <int S>
constexpr GreedyOrder greedy_order()
{
    GreedyOrder o{{0, 0}, 0};
    greedy_visit(o, 0, S - 1);
    return o;
}

// Limbs of the exact sums behind floor(T) (exact_floor_t below): value = sum_i limb[i] * 2^(32 i - 149).  An fp32 value
// starts in limb 7 at the latest and touches three limbs; what the 64 bits of the top limb hold beyond 32 is headroom
// for the sum and the coefficients, and the carry out of it gives the sign.
constexpr int kExactLimbs = 10;

// LDS of one bucket: D = element capacity, B = number of bins.
template <int D_, int B_, int S_>
struct alignas(16) OrqLds {
    static constexpr int D = D_, B = B_;
    static constexpr int BLOCK = D_ / 64;  // positions per entry of the fp64 block prefix
    uint32_t grouped[D];  // fp32 bit patterns grouped by bin (-0 lies with +0), unsorted inside a bin
    uint32_t bin_start[B + 1];  // histogram, then first position of each bin; [B] = bucket length
    double block_prefix[64];    // fp64 sum of all positions before block l (block = D/64 positions)
    // per level k: value; #{v < value}; #{v <= value}; sum{v < value}; sum{v <= value}; the rank it
    // was picked at (0 = not picked by rank)
    double lvl_sum_lt[S_];
    double lvl_sum_le[S_];
    float lvl_value[S_];
    uint32_t lvl_count_lt[S_];
    uint32_t lvl_count_le[S_];
    uint32_t lvl_rank[S_];
    double sum_error_bound;  // 0 when every fp64 sum of the bucket is exact (see floor_t_from_sums)
    unsigned long long exact_limb[1][kExactLimbs];  // workspace of exact_floor_t
};

// A zero the compiler cannot see through.  x + this turns -0 into +0 like x + 0.0f does, and, unlike that, is not
// recognised as the same value in a later phase: what is derived from the register-resident bucket is computed again
// where it is needed instead of being kept in registers (and no copy of x is made to hide it).
__device__ __forceinline__ float opaque_zero()
{
    float zero = 0.0f;
    asm volatile("" : "+v"(zero));
    return zero;
}

// What the histogram keeps per element: the element's position inside its bin in the upper half, and in the lower half
// the byte offset of its bin's counter from the middle of the bin table (signed, at most +-4096: the low half of the
// very register that addressed the returning add; one byte permute packs the two).
__device__ __forceinline__ uint32_t pack_slot(uint32_t position_in_bin, uint32_t bin, uint32_t half)
{
    return __builtin_amdgcn_perm(position_in_bin, (bin - half) * 4u, 0x05040100u);
}

// First position of the slot's bin: table = the middle of the bin-start table (one sign-extending bit-field extract).
template <class T>
__device__ __forceinline__ uint32_t slot_bin_start(const T* table_middle, uint32_t slot)
{
    const int32_t byte_offset = (int32_t)(int16_t)(slot & 0xFFFFu);
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(table_middle) + byte_offset);
}

__device__ __forceinline__ uint32_t umin32(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ __forceinline__ uint32_t umax32(uint32_t a, uint32_t b) { return a > b ? a : b; }

// Bin of a value (with -0 already turned into +0): the HALF bins of either sign cover 16 binades below the
// largest magnitude of the bucket (t_low = its lowest regular bin index); everything smaller shares the two
// centre bins HALF - 1 and HALF.  The upper clamp only acts on NaN.
template <int HALF, int SHIFT>
__device__ __forceinline__ uint32_t value_bin(float canonical, uint32_t t_low)
{
    const uint32_t bits = __float_as_uint(canonical);
    const uint32_t t = (bits & 0x7FFFFFFFu) >> SHIFT;
    const uint32_t u = umin32(__builtin_elementwise_sub_sat(t, t_low), (uint32_t)(HALF - 1));  // 0 .. HALF-1
    const uint32_t negative = (uint32_t)((int32_t)bits >> 31);                                 // 0 or ~0
    return (uint32_t)HALF + (u ^ negative);  // HALF + u, or HALF - 1 - u for a negative value
}

// Sort key of a value as stored in the grouped array (bit pattern of the element; -0 counts as +0).
__device__ __forceinline__ uint32_t stored_key(uint32_t stored) { return float_to_key(__uint_as_float(stored) + 0.0f); }

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x)
{
    x = umax32(x, dpp_u32<kDppXor1>(x));
    x = umax32(x, dpp_u32<kDppXor2>(x));
    x = umax32(x, dpp_u32<kDppHalfMirror>(x));
    x = umax32(x, dpp_u32<kDppMirror>(x));
    return umax32(umax32(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
                  umax32(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) { return ~wave_max_u32(~x); }

// Inclusive scans over the lanes in ascending lane order, in registers: four shifts inside every row of 16
// lanes (a lane without a source adds 0), then the last lane of row 0 / 2 is added to row 1 / 3 and lane 31
// to the upper half (DPP row_shr, row_bcast:15, row_bcast:31).
constexpr int kDppRowShr1 = 0x111, kDppRowShr2 = 0x112, kDppRowShr8 = 0x118, kDppRowBcast15 = 0x142,
              kDppRowBcast31 = 0x143;

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_zero_u32(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROW_MASK, 0xF, false);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_or_zero_f64(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = dpp_or_zero_u32<CTRL, ROW_MASK>((uint32_t)u), hi = dpp_or_zero_u32<CTRL, ROW_MASK>((uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ uint32_t wave_inclusive_scan_u32(uint32_t x)
{
    x += dpp_or_zero_u32<kDppRowShr1, 0xF>(x);
    x += dpp_or_zero_u32<kDppRowShr2, 0xF>(x);
    x += dpp_or_zero_u32<kDppRowShr4, 0xF>(x);
    x += dpp_or_zero_u32<kDppRowShr8, 0xF>(x);
    x += dpp_or_zero_u32<kDppRowBcast15, 0xA>(x);
    x += dpp_or_zero_u32<kDppRowBcast31, 0xC>(x);
    return x;
}

__device__ __forceinline__ double wave_inclusive_scan_f64(double x)
{
    x += dpp_or_zero_f64<kDppRowShr1, 0xF>(x);
    x += dpp_or_zero_f64<kDppRowShr2, 0xF>(x);
    x += dpp_or_zero_f64<kDppRowShr4, 0xF>(x);
    x += dpp_or_zero_f64<kDppRowShr8, 0xF>(x);
    x += dpp_or_zero_f64<kDppRowBcast15, 0xA>(x);
    x += dpp_or_zero_f64<kDppRowBcast31, 0xC>(x);
    return x;
}

// Ascending bitonic sorts in registers.  Every compare-exchange is ascending: the first step of a merge pairs
// element e with e ^ (run length - 1), i.e. meets the second run in reverse, the others pair e with e ^ J; the lane
// whose bit (run length / 2, or J) is clear keeps the smaller key.  So no step needs a direction, a step is one
// cross-lane move and one median of three, and every row of 16 lanes (half of the wavefront) is sorted ascending
// on its own after 10 (15) of the 21 steps.
constexpr int kDppQuadReverse = 0x1B;  // quad_perm [3,2,1,0]: partner lane ^ 3

// Value held by lane (lane ^ (2 M - 1)): every group of 2 M lanes in reverse order.
template <int M>
__device__ __forceinline__ uint32_t lane_reverse(uint32_t x, uint32_t lane)
{
    if constexpr (M == 1) {
        return dpp_u32<kDppXor1>(x);
    } else if constexpr (M == 2) {
        return dpp_u32<kDppQuadReverse>(x);
    } else if constexpr (M == 4) {
        return dpp_u32<kDppHalfMirror>(x);
    } else if constexpr (M == 8) {
        return dpp_u32<kDppMirror>(x);
    } else if constexpr (M == 16) {
        return lane_xor<16>(dpp_u32<kDppMirror>(x), lane);
    } else {
        static_assert(M == 32, "groups of at most 64 lanes");
        return lane_xor<32>(lane_xor<16>(dpp_u32<kDppMirror>(x), lane), lane);
    }
}

// Median of three (v_med3_u32): with bound = 0 the smaller, with bound = 0xFFFFFFFF the larger of x and y.
__device__ __forceinline__ uint32_t smaller_or_larger(uint32_t x, uint32_t y, uint32_t bound)
{
    return umax32(umin32(x, y), umin32(umax32(x, y), bound));
}

// 0 in the lanes whose bit BIT is clear (they keep the smaller key of a pair), 0xFFFFFFFF in the others.
template <int BIT>
__device__ __forceinline__ uint32_t upper_lanes(uint32_t lane)
{
    return (lane & (uint32_t)BIT) ? 0xFFFFFFFFu : 0u;
}

// One key per lane: merges sorted runs of M lanes into runs of 2 M.
template <int M>
__device__ __forceinline__ uint32_t wave_sort_merge(uint32_t x, uint32_t lane)
{
    x = smaller_or_larger(x, lane_reverse<M>(x, lane), upper_lanes<M>(lane));
    if constexpr (M >= 32) x = smaller_or_larger(x, lane_xor<16>(x, lane), upper_lanes<16>(lane));
    if constexpr (M >= 16) x = smaller_or_larger(x, lane_xor<8>(x, lane), upper_lanes<8>(lane));
    if constexpr (M >= 8) x = smaller_or_larger(x, lane_xor<4>(x, lane), upper_lanes<4>(lane));
    if constexpr (M >= 4) x = smaller_or_larger(x, lane_xor<2>(x, lane), upper_lanes<2>(lane));
    if constexpr (M >= 2) x = smaller_or_larger(x, lane_xor<1>(x, lane), upper_lanes<1>(lane));
    return x;
}

// `count` lanes (the first ones) hold keys, the others 0xFFFFFFFF: with at most 16 (32) keys only the first
// row (half) of the wavefront has to be sorted.
__device__ __forceinline__ uint32_t wave_sort_u32(uint32_t x, uint32_t lane, uint32_t count)
{
    x = wave_sort_merge<1>(x, lane);
    x = wave_sort_merge<2>(x, lane);
    x = wave_sort_merge<4>(x, lane);
    x = wave_sort_merge<8>(x, lane);
    if (count <= 16u) return x;
    x = wave_sort_merge<16>(x, lane);
    if (count <= 32u) return x;
    return wave_sort_merge<32>(x, lane);
}

// The key of 1-based rank `rank` among the first `count` (at most 64) lanes' keys, the other lanes holding 0xFFFFFFFF;
// the answer is known to sit in one of the lanes `open`.  count_le = number of keys not above it; returns the lanes with
// smaller keys.
//
// Quickselect on lane masks: a pivot costs one lane read and two compares on the vector unit, counting and narrowing are
// scalar.  A bin of 20 keys takes about 5 pivots, i.e. 15 vector instructions where a bitonic sort of the keys takes 42
// (65 above 32 keys), which the issue of vector instructions bound; what a solve now waits for is the pivots' scalar chain.
// The pivot is the first open lane at or above lane rank - 1: the answer itself when the keys came in sorted.  Every round
// drops the pivot at least, so the loop ends.  In assembly because the compiler spends twice the scalar instructions on it.  Wait states: two
// between the lane read and the compares that take the key (s_nop 1); three scalar instructions lie between whatever
// wrote `mine` and the lane read.  All lanes are active.
__device__ __forceinline__ uint64_t select_rank(uint32_t mine, uint32_t count, uint32_t rank, uint64_t open, uint32_t& key_out,
                                                uint32_t& count_le_out)
{
    const uint64_t valid = ~0ull >> (64u - count);  // (count >= 1)
    const uint64_t from_rank = ~0ull << (rank - 1u);
    uint32_t key, pivot, count_lt, count_le;
    uint64_t lt, le;
    asm("1:\n\t"
        "s_and_b64 %[le], %[open], %[from]\n\t"
        "s_cselect_b64 %[le], %[le], %[open]\n\t"
        "s_ff1_i32_b64 %[pivot], %[le]\n\t"
        "v_readlane_b32 %[key], %[mine], %[pivot]\n\t"
        "s_nop 1\n\t"
        "v_cmp_gt_u32_e64 %[lt], %[key], %[mine]\n\t"
        "v_cmp_ge_u32_e64 %[le], %[key], %[mine]\n\t"
        "s_bcnt1_i32_b64 %[count_lt], %[lt]\n\t"
        "s_and_b64 %[le], %[le], %[valid]\n\t"
        "s_bcnt1_i32_b64 %[count_le], %[le]\n\t"
        "s_cmp_le_u32 %[rank], %[count_lt]\n\t"
        "s_cbranch_scc1 2f\n\t"
        "s_cmp_le_u32 %[rank], %[count_le]\n\t"
        "s_cbranch_scc1 3f\n\t"
        "s_andn2_b64 %[open], %[open], %[le]\n\t"
        "s_cbranch_scc1 1b\n\t"
        "s_branch 3f\n"
        "2:\n\t"
        "s_and_b64 %[open], %[open], %[lt]\n\t"
        "s_cbranch_scc1 1b\n"
        "3:"
        : [open] "+&s"(open), [key] "=&s"(key), [pivot] "=&s"(pivot), [count_lt] "=&s"(count_lt), [count_le] "=&s"(count_le),
          [lt] "=&s"(lt), [le] "=&s"(le)
        : [mine] "v"(mine), [rank] "s"(rank), [valid] "s"(valid), [from] "s"(from_rank)
        : "scc");
    key_out = key;
    count_le_out = count_le;
    return lt;
}

// The bucket element of a given rank, with the counts and sums of the bucket elements strictly
// below it and not above it.
struct Picked {
    uint32_t key;
    uint32_t count_lt, count_le;
    double sum_lt, sum_le;
};

// The element of 1-based rank `rank`, which lies in the bin that holds positions [first, first + count).  BLOCK =
// positions per entry of the fp64 block prefix (at most 64).
// SUMS = false: only the element is wanted (rules whose solves never read the counts and sums of a picked level: a
// single interior level, Linear-s); the block prefix is then neither needed nor read.
template <int BLOCK, bool SUMS = true, class Lds>
__device__ __forceinline__ Picked pick_in_span(const Lds& lds, uint32_t first, uint32_t count, uint32_t rank, uint32_t lane)
{
    static_assert(BLOCK <= 64, "the head of a block is read one position per lane");
    // The sum of everything before the bin is the prefix of its block plus the block's positions before `first` (the
    // bin's "front").  Front and bin are neighbours in the grouped array, and every key of the front is smaller: where
    // the two fit the lanes they are read, ranked and summed as one.
    const uint32_t block = first / BLOCK;
    const uint32_t front = SUMS ? first - block * BLOCK : 0u;
    double before_block = 0.0;
    if constexpr (SUMS) before_block = lds.block_prefix[block];

    uint32_t key, c_lt, c_le;  // counts from the bin's first position on
    double s_lt;
    if (count <= 64u) {
        const uint32_t joint = front + count <= 64u ? front : 0u;  // lanes that hold the front
        const uint32_t held = joint + count;
        const float value =
            __uint_as_float(lds.grouped[first - joint + (lane < held ? lane : 0u)]) + 0.0f;
        const uint32_t mine = lane < held ? float_to_key(value) : 0xFFFFFFFFu;
        float other = 0.0f;  // the front where it does not fit
        if (SUMS && joint != front) other = lane < front ? __uint_as_float(lds.grouped[first - front + lane]) : 0.0f;
        const uint64_t lt =
            select_rank(mine, held, rank - first + joint, (~0ull >> (64u - count)) << joint, key, c_le);
        c_le -= joint;
        c_lt = (uint32_t)__popcll(lt) - joint;
        if constexpr (SUMS) {
            double part = __builtin_amdgcn_inverse_ballot_w64(lt) ? (double)value : 0.0;
            if (joint != front) part += (double)other;
            s_lt = wave_sum(part);
        } else {
            s_lt = 0.0;
        }
    } else {
        const uint32_t r_in = rank - first;  // 1-based rank inside the bin
        const float head = lane < front ? __uint_as_float(lds.grouped[first - front + lane]) : 0.0f;
        // A crowded bin (many equal or nearly equal values): bisection on the key, over the bits in which the bin's
        // smallest and largest key differ (none when all its values are equal).  Up to 256 keys stay in registers.
        constexpr int HELD = 4;
        const bool held = count <= 64u * HELD;
        uint32_t mine[HELD];
        uint32_t smallest = 0xFFFFFFFFu, largest = 0u;
        if (held) {
#pragma unroll
            for (int c = 0; c < HELD; ++c) {
                const uint32_t i = 64u * c + lane;
                const bool valid = i < count;
                mine[c] = valid ? stored_key(lds.grouped[first + (valid ? i : 0u)]) : 0xFFFFFFFFu;
                smallest = umin32(smallest, mine[c]);
                largest = umax32(largest, valid ? mine[c] : 0u);
            }
        } else {
            for (uint32_t base = 0; base < count; base += 64u) {
                const uint32_t i = base + lane;
                if (i < count) {
                    const uint32_t k = stored_key(lds.grouped[first + i]);
                    smallest = umin32(smallest, k);
                    largest = umax32(largest, k);
                }
            }
        }
        smallest = wave_min_u32(smallest);
        largest = wave_max_u32(largest);
        const uint32_t differing = smallest ^ largest;
        uint32_t prefix = smallest;
        if (differing != 0u) {
            const int top = 31 - __builtin_clz(differing);
            prefix = top == 31 ? 0u : smallest & ~((2u << top) - 1u);  // the bits above `top` are common to all keys
            for (int bit = top; bit >= 0; --bit) {
                const uint32_t cand = prefix | (1u << bit);
                uint32_t below = 0;
                if (held) {
#pragma unroll
                    for (int c = 0; c < HELD; ++c) below += (uint32_t)__popcll(__ballot(mine[c] < cand));
                } else {
                    for (uint32_t base = 0; base < count; base += 64u) {
                        const uint32_t i = base + lane;
                        const uint32_t k = i < count ? stored_key(lds.grouped[first + i]) : 0xFFFFFFFFu;
                        below += (uint32_t)__popcll(__ballot(k < cand));
                    }
                }
                if (below < r_in) prefix = cand;
            }
        }
        key = prefix;
        c_lt = 0;
        c_le = 0;
        double part = (double)head;
        if constexpr (SUMS)
        for (uint32_t base = 0; base < count; base += 64u) {
            const uint32_t i = base + lane;
            const float x = i < count ? __uint_as_float(lds.grouped[first + i]) + 0.0f : 0.0f;
            const uint32_t k = i < count ? float_to_key(x) : 0xFFFFFFFFu;
            const bool lt = k < key;
            c_lt += (uint32_t)__popcll(__ballot(lt));
            c_le += (uint32_t)__popcll(__ballot(k <= key && i < count));
            part += lt ? (double)x : 0.0;
        }
        s_lt = SUMS ? wave_sum(part) : 0.0;
    }
    Picked p;
    p.key = key;
    p.count_lt = first + c_lt;
    p.count_le = first + c_le;
    p.sum_lt = before_block + s_lt;
    const uint32_t equal = c_le - c_lt;
    double equal_sum = (double)key_to_float(key);
    if (equal != 1u) equal_sum *= (double)equal;
    p.sum_le = p.sum_lt + equal_sum;
    return p;
}

// The same for bin `bin`.
template <int BLOCK, bool SUMS = true, class Lds>
__device__ __forceinline__ Picked pick_in_bin(const Lds& lds, uint32_t bin, uint32_t rank, uint32_t lane)
{
    const uint32_t first = uniform_u32(lds.bin_start[bin]);
    const uint32_t count = uniform_u32(lds.bin_start[bin + 1]) - first;
    return pick_in_span<BLOCK, SUMS>(lds, first, count, rank, lane);
}

// rank is 1-based, 1 <= rank <= bucket length.  my_start[t] = bin_start[lane * PER + t], kept in registers.
template <int D, int B, int S, bool SUMS = true>
__device__ __forceinline__ Picked pick_rank(const OrqLds<D, B, S>& lds, const uint32_t (&my_start)[B / 64],
                                            uint32_t rank, uint32_t lane)
{
    constexpr int PER = B / 64;
    // the bin holding the rank: the last bin whose first position is below the rank (counted on the scalar unit)
    uint32_t starts_below = 0;
#pragma unroll
    for (int t = 0; t < PER; ++t) starts_below += (uint32_t)__popcll(__ballot(my_start[t] < rank));
    const uint32_t bin = starts_below - 1u;  // bin_start[0] = 0 < rank: at least one
    return pick_in_bin<D / 64, SUMS>(lds, bin, rank, lane);
}

// The same with the bin found by two looks into LDS (every (B/64)-th bin start, then the B/64 bins in between):
// no registers are tied up by the bin starts.
template <bool SUMS = true, class Lds>
__device__ __forceinline__ Picked pick_rank_by_lookup(const Lds& lds, uint32_t rank, uint32_t lane)
{
    constexpr uint32_t PER = Lds::B / 64;
    static_assert(PER <= 64, "one lane per bin of a segment");
    const uint32_t coarse = lds.bin_start[lane * PER];
    const uint32_t segment = (uint32_t)__popcll(__ballot(coarse < rank)) - 1u;
    const uint32_t fine = lds.bin_start[segment * PER + (lane < PER ? lane : 0u)];
    const uint32_t within = (uint32_t)__popcll(__ballot(lane < PER && fine < rank)) - 1u;  // the bin is segment * PER + within
    // its first position and that of the next bin are already in the registers of two lanes
    const uint32_t first = __builtin_amdgcn_readlane(fine, within);
    const uint32_t next = within + 1u < PER ? __builtin_amdgcn_readlane(fine, (within + 1u) & 63u)
                          : segment < 63u   ? __builtin_amdgcn_readlane(coarse, (segment + 1u) & 63u)
                                            : uniform_u32(lds.bin_start[Lds::B]);
    return pick_in_span<Lds::BLOCK, SUMS>(lds, first, next - first, rank, lane);
}

// ----------------------------------------------------------------------------------------------
// floor(T) of the discrete optimal condition (second remark after Theorem 1), T = S / (R - L) with
// S = sum over the bucket elements v in [L, R] of (v - L).  The floor decides which element becomes the level, so it
// is the exact one: the largest integer m with S - m (R - L) >= 0.
//
// Fast path.  The sums a solve reads are fp64 sums of fp32 values.  They are exact, whatever their order, when every
// non-zero element of the bucket is at most safe_binades(len) binades below the largest magnitude M < 2^(E+1): every
// element is then a multiple of q = 2^(E - safe - 23), every intermediate value (prefix sums below len * M; their
// differences, S and m (R - L) below 2 len M < len * 2^(E+2)) is a multiple of q below 2^53 q, so no addition,
// difference or product ever rounds.  With
// S exact, floor(S / (R - L)) is corrected by at most one through the sign of the exact rest S - m (R - L).  A bucket
// with smaller non-zero elements ("tiny" ones: they sit in the two centre bins of the grouping) keeps the same
// arithmetic, but a rest within sum_error_bound of 0 or of R - L does not decide; the bound covers 256 roundings of
// half a unit in the last place of a value below 2 len M, more than any prefix sum here goes through.
//
// Exact path (undecided solves only).  Every fp32 value is an integer multiple of 2^-149: the elements in [L, R] are
// added up as signed fixed-point numbers in 10 limbs of 32 payload bits (64-bit LDS atomics; a limb takes at most
// 32768 pieces below 2^32 before the carries are propagated), and m is searched with the sign of
// sum - (c - m) L - m R, c the number of elements in [L, R], which does not grow with m.
// ----------------------------------------------------------------------------------------------

__host__ __device__ constexpr uint32_t ceil_log2(uint32_t n)
{
    uint32_t k = 0;
    while ((1u << k) < n) ++k;
    return k;
}

// How many binades below the largest magnitude a non-zero element may lie for all fp64 sums of a bucket of at most
// `capacity` elements to be exact: capacity * 2 M / q < 2^53 with q = 2^(E - safe - 23) and M < 2^(E+1).
__host__ __device__ constexpr uint32_t safe_binades(uint32_t capacity) { return 28u - ceil_log2(capacity); }

// What the fp64 sums of a bucket with tiny elements can be off by: 2^(ceil_log2(capacity) + E - 44), E the
// unbiased exponent of the largest magnitude (at least the smallest normal double).
__device__ __forceinline__ double sum_error_bound_of(uint32_t mag_max_bits, uint32_t capacity)
{
    const int field = 1023 + ((int)(mag_max_bits >> 23) - 127) + (int)ceil_log2(capacity) - 44;
    return __longlong_as_double((long long)(uint64_t)(field < 1 ? 1 : field) << 52);
}

// Cuts |c * v| into the three 32-bit pieces that go to limbs first, first + 1, first + 2.  first <= 7.
struct ExactPieces {
    uint32_t first;
    bool negative;
    uint64_t piece[3];
};

__device__ __forceinline__ ExactPieces exact_pieces(float v, long long c)
{
    const uint32_t bits = __float_as_uint(v);
    const uint32_t biased = (bits >> 23) & 0xFFu, fraction = bits & 0x7FFFFFu;
    // |v| = mantissa * 2^(position - 149); subnormals have position 0 and no hidden bit
    const uint64_t mantissa = biased ? (fraction | 0x800000u) : fraction;
    const uint32_t position = biased ? biased - 1u : 0u;
    const uint64_t magnitude = mantissa * (uint64_t)(c < 0 ? -c : c);  // below 2^44
    const uint32_t shift = position & 31u;
    const uint64_t low = magnitude << shift;                          // bits 0 .. 63 of magnitude << shift
    const uint64_t high = shift > 20u ? magnitude >> (64u - shift) : 0ull;  // bits 64 .. 74
    ExactPieces p;
    p.first = position >> 5;
    p.negative = ((bits >> 31) != 0u) != (c < 0);
    p.piece[0] = low & 0xFFFFFFFFull;
    p.piece[1] = low >> 32;
    p.piece[2] = high;
    return p;
}

// limb (LDS, shared by the lanes of the group) += v
__device__ __forceinline__ void exact_add_shared(unsigned long long* limb, float v)
{
    const ExactPieces p = exact_pieces(v, 1);
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (p.piece[k] != 0ull) atomicAdd(&limb[p.first + k], p.negative ? 0ull - p.piece[k] : p.piece[k]);  // signed, mod 2^64
}

// The piece of p that belongs to limb i.
__device__ __forceinline__ long long exact_piece_of(const ExactPieces& p, uint32_t i)
{
    const uint32_t k = i - p.first;  // 0, 1, 2 for the three limbs the value touches
    const uint64_t piece = k == 0u ? p.piece[0] : k == 1u ? p.piece[1] : k == 2u ? p.piece[2] : 0ull;
    return p.negative ? -(long long)piece : (long long)piece;
}

// sum (the limbs) + cl * L + cr * R >= 0 ?  The limbs are only read.  (A rolled loop over the limbs: this rare path
// must not raise the register count of the kernels it is inlined into.)
__device__ __forceinline__ bool exact_not_negative(const unsigned long long* limb, float L, long long cl, float R,
                                                   long long cr)
{
    const ExactPieces pl = exact_pieces(L, cl), pr = exact_pieces(R, cr);
    long long carry = 0;
#pragma unroll 1
    for (uint32_t i = 0; i < (uint32_t)kExactLimbs; ++i) {
        const long long t = (long long)limb[i] + exact_piece_of(pl, i) + exact_piece_of(pr, i) + carry;
        carry = t >> 32;  // floor division by 2^32
    }
    return carry >= 0;  // what is left above the top limb carries the sign
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// floor(T), exactly.  Called by all lanes that hold the bucket (a wavefront, or the group of lanes of a small bucket)
// with the same limb array, L < R, count_in = #{L <= v <= R} and a first guess; each_of_mine(f) runs f(x) on the bucket
// elements this lane answers for; lane_in_group counts the calling lanes from 0.
template <class EachFn>
__device__ __forceinline__ uint32_t exact_floor_t(unsigned long long* limb, uint32_t lane_in_group, float L, float R,
                                                  uint32_t count_in, uint32_t guess, EachFn each_of_mine)
{
    if (lane_in_group < (uint32_t)kExactLimbs) limb[lane_in_group] = 0ull;
    wave_lds_sync();
    each_of_mine([&](float x) {
        if (L <= x && x <= R) exact_add_shared(limb, x);
    });
    wave_lds_sync();
    // S - m (R - L) = sum - (count_in - m) L - m R; the first two probes sit at the guess
    uint32_t lo = 0u, hi = count_in;  // m = 0 fits: S >= 0
    uint32_t probe = guess < count_in ? guess : count_in;
    if (probe == 0u) probe = hi > 0u ? 1u : 0u;
    for (int step = 0; lo < hi; ++step) {
        const uint32_t mid = step == 0 ? probe : (step == 1 && lo == probe && probe < hi) ? probe + 1u
                                                                                         : lo + (hi - lo + 1u) / 2u;
        if (exact_not_negative(limb, L, -(long long)(count_in - mid), R, -(long long)mid)) lo = mid;
        else hi = mid - 1u;
    }
    wave_lds_sync();  // every lane is through with the limbs before a later call clears them
    return lo;
}

// The two forms the kernels call, as real functions: inlined into every level solve, this rare path cost the kernels
// 3 to 20 % of their speed (code size, registers) without ever running.
//   bucket grouped in LDS: the calling lanes take the positions lane, lane + stride, ... below len
static __device__ __attribute__((noinline)) uint32_t exact_floor_t_grouped(unsigned long long* limb, const uint32_t* grouped,
                                                                   uint32_t len, uint32_t lane, uint32_t stride, float L,
                                                                   float R, uint32_t count_in, uint32_t guess)
{
    return exact_floor_t(limb, lane, L, R, count_in, guess, [&](auto add) {
        for (uint32_t i = lane; i < len; i += stride) add(__uint_as_float(grouped[i]));
    });
}

//   small bucket in registers: every lane of the bucket's group brings four elements, `valid` of which exist
static __device__ __attribute__((noinline)) uint32_t exact_floor_t_registers(unsigned long long* limb, uint32_t lane_in_group,
                                                                     float L, float R, uint32_t count_in, uint32_t guess,
                                                                     float x0, float x1, float x2, float x3, uint32_t valid)
{
    return exact_floor_t(limb, lane_in_group, L, R, count_in, guess, [&](auto add) {
        if (valid > 0u) add(x0);
        if (valid > 1u) add(x1);
        if (valid > 2u) add(x2);
        if (valid > 3u) add(x3);
    });
}

// floor(T) of one solve from the fp64 sums (see above): Ssum = the sums' S, width = R - L > 0 in fp64, bound = the
// bucket's sum_error_bound (0: every sum is exact).  Returns false when the sums do not decide; m is then the guess for
// exact_floor_t.  The quotient only proposes m (a reciprocal and a product instead of a division: any m whose rest
// S - m width lies inside (bound, width - bound) is the floor); the common case costs the reciprocal, a product, a
// floor, a fused multiply-add for the rest and two comparisons.  A rest of exactly 0 (T an integer) or outside
// [0, width) takes the second branch, which moves m by one where the quotient's rounding asks for it.
__device__ __forceinline__ bool floor_t_from_sums(double Ssum, double width, double bound, double& m)
{
    m = fmax(floor(Ssum * __builtin_amdgcn_rcp(width)), 0.0);  // (NaN from non-finite input becomes 0)
    double rest = __builtin_fma(-m, width, Ssum);  // exact when bound == 0: m * width has at most 41 bits
    if (rest > bound && width - rest > bound) return true;
    if (rest < 0.0) {
        m = fmax(m - 1.0, 0.0);
        rest = __builtin_fma(-m, width, Ssum);
    } else if (rest >= width) {
        m += 1.0;
        rest = __builtin_fma(-m, width, Ssum);
    }
    if (bound == 0.0) return true;  // exact sums, exact rest: 0 <= rest < width now
    return rest > bound && width - rest > bound;
}

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr float kNoElement = __builtin_nanf("");  // what a wavefront holds in place of elements past a range's end

// Runs f(c, all) for the chunks c (256 elements each) that hold at least one of the `len` valid elements.  `all` is a
// std::true_type when every element of the chunk is valid, so that f can drop its per-element bounds tests: at most one
// chunk of a bucket is cut by its end, and the chunks past it are skipped altogether (wave-uniform branches).
template <int C, bool FULL, class F>
__device__ __forceinline__ void for_each_chunk(uint32_t len, F f)
{
#pragma unroll
    for (int c = 0; c < C; ++c) {
        if (FULL || 256u * (uint32_t)(c + 1) <= len) f(c, std::true_type{});
        else if (256u * (uint32_t)c < len) f(c, std::false_type{});
    }
}

// ---- encode (random rounding, Section 3.1) + pack ------------------------------------------------
// Interval of an element among S levels: the last level not above it, at most S - 2.  base = that level, width = the next
// one minus it (fp32, one rounding), bit[p] = lanes whose interval index has bit p set.  Up to four levels one compare per
// interior level; from five levels on a binary search, whose compare masks are the index bits: with eight levels 13
// vector instructions per element instead of the 18 of one compare and two selects per interior level, with nine 14
// instead of 21.
template <int S>
struct Interval {
    static constexpr int kIndexBits = S == 2 ? 0 : S == 3 ? 1 : S <= 5 ? 2 : 3;
    float base, width;
    uint64_t bit[3];
};

template <int S>
__device__ __forceinline__ Interval<S> find_interval(float x, const float (&lv)[S], const float (&width)[S - 1])
{
    static_assert((S >= 2 && S <= 5) || S == 8 || S == 9, "level counts of the schemes");
    Interval<S> r;
    if constexpr (S <= 4) {
        r.base = lv[0];
        r.width = width[0];
        uint64_t not_below[3] = {0, 0, 0};  // [t]: lanes whose element is not below level t, t = 1 .. S - 2
#pragma unroll
        for (int t = 1; t < S - 1; ++t) {
            const bool ge = lv[t] <= x;
            not_below[t] = __ballot(ge);
            // (values, not a choice between two objects: that one is compiled to an address in scratch memory)
            const float base = lv[t], above = width[t], old_base = r.base, old_width = r.width;
            r.base = ge ? base : old_base;
            r.width = ge ? above : old_width;
        }
        r.bit[0] = not_below[1] ^ not_below[2];
        r.bit[1] = not_below[2];
    } else if constexpr (S == 5) {
        const bool m1 = lv[2] <= x;
        const float t = m1 ? lv[3] : lv[1];
        const bool m0 = t <= x;
        const float low = m1 ? lv[2] : lv[0], high = m1 ? lv[4] : lv[2];
        r.base = m0 ? t : low;
        r.width = (m0 ? high : t) - r.base;
        r.bit[0] = __ballot(m0);
        r.bit[1] = __ballot(m1);
    } else {
        const bool m2 = lv[4] <= x;
        const float t1 = m2 ? lv[6] : lv[2];
        const bool m1 = t1 <= x;
        const float low7 = m2 ? lv[7] : lv[3], low5 = m2 ? lv[5] : lv[1];
        const float t0 = m1 ? low7 : low5;
        r.bit[2] = __ballot(m2);
        r.bit[1] = __ballot(m1);
        r.bit[0] = __ballot(t0 <= x);
        if constexpr (S == 8) r.bit[0] &= ~(r.bit[1] & r.bit[2]);  // the top level begins no interval
        const bool m0 = __builtin_amdgcn_inverse_ballot_w64(r.bit[0]);
        const float low = m2 ? lv[4] : lv[0];
        const float even = m1 ? t1 : low;
        const float next_of_3 = S == 9 ? (m2 ? lv[S - 1] : lv[4]) : lv[4];
        const float next = m1 ? next_of_3 : t1;
        r.base = m0 ? t0 : even;
        r.width = (m0 ? next : t0) - r.base;
    }
    return r;
}

// 2 x + (1 in the lanes of `mask`), as one add with carry (the compiler makes a select and a shift-and-or of it).
// RAW: the mask comes straight from a vector compare, which needs two wait states before a vector instruction reads it
// (the compiler does not look into the asm); a mask computed on the scalar unit needs none.
template <bool RAW>
__device__ __forceinline__ uint32_t push_bit(uint32_t x, uint64_t mask)
{
    uint32_t r;
    uint64_t carry_out;
    if constexpr (RAW) asm("s_nop 1\n\tv_addc_co_u32_e64 %0, %1, %2, %2, %3" : "=v"(r), "=s"(carry_out) : "v"(x), "s"(mask));
    else asm("v_addc_co_u32_e64 %0, %1, %2, %2, %3" : "=v"(r), "=s"(carry_out) : "v"(x), "s"(mask));
    return r;
}

// x = 2 x + (1 in the lanes where a < b), y likewise: two compares, two wait states (the compiler does not look into the asm), two adds with carry; one
// pair's instructions are most of the other's wait.
__device__ __forceinline__ void push_less(uint32_t& x, float a, float b, uint32_t& y, float c, float d)
{
    uint64_t first, second;
    asm("v_cmp_lt_f32_e64 %2, %4, %5\n\tv_cmp_lt_f32_e64 %3, %6, %7\n\ts_nop 0\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %2\n\tv_addc_co_u32_e64 %1, vcc, %1, %1, %3"
        : "+v"(x), "+v"(y), "=&s"(first), "=&s"(second)
        : "v"(a), "v"(b), "v"(c), "v"(d)
        : "vcc");
}

// The largest number below x (x finite).
__device__ __forceinline__ float next_below(float x)
{
    const uint32_t u = __float_as_uint(x);
    return __uint_as_float((u << 1) == 0u ? 0x80000001u : (u >> 31) != 0u ? u + 1u : u - 1u);
}

// How the elements a wavefront encodes lie in its registers.  kBlocks: Philox blocks from chunk to chunk.  group, half:
// which half of which 64-element group the lanes 8 h .. 8 h + 7 hold of chunk c; row_groups =
// 64-element groups from row to row.
//   OneRange: chunk c, lane l: elements 256c + 4l + {0..3} of one range.
//   Rows<LANES>: every row of LANES = 16 or 8 lanes holds a range of its own (consecutive ranges of equal length), chunk c, lane i of
//                the row: elements 4 LANES c + 4i + {0..3} of that range.
struct OneRange {
    static constexpr uint32_t kBlocks = 64;
    static __device__ __forceinline__ uint32_t group(uint32_t c, uint32_t h, uint32_t row_groups) { return 4u * c + (h >> 1) * row_groups; }
    static __device__ __forceinline__ uint32_t half(uint32_t, uint32_t h) { return h & 1u; }
};
template <int LANES>
struct Rows {
    static_assert(LANES == 16 || LANES == 8, "a chunk of a row is 64 or 32 elements");
    static constexpr uint32_t kBlocks = LANES;
    static __device__ __forceinline__ uint32_t group(uint32_t c, uint32_t h, uint32_t row_groups)
    {
        return LANES == 16 ? c + (h >> 1) * row_groups : (c >> 1) + h * row_groups;
    }
    static __device__ __forceinline__ uint32_t half(uint32_t c, uint32_t h) { return (LANES == 16 ? h : c) & 1u; }
};

// LDS through its own address space: addresses of 32 bits.
typedef __attribute__((address_space(3))) uint32_t LdsWord;
typedef __attribute__((address_space(3))) uint16_t LdsHalf;
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) floatx2 LdsPair;

// Where the encoder may keep its levels in LDS: `table` = LDS address of S - 1 pairs (level k, the width above it) for the ranges
// of this lane, 8-byte aligned; `writer`: one lane per table.
struct PairsInLds {
    static constexpr bool kUsed = true;
    uint32_t table;
    bool writer;
};
struct NoPairs {
    static constexpr bool kUsed = false;
};

// Which of the chunks' elements exist: all; those below `len`; or all of the chunks below len / 256.  Those that do not
// exist in a chunk that does are NaN: no comparison with NaN holds, so their bits come out as 0.
enum class Fill { kAll, kRagged, kWholeChunks };

// The encoder's random numbers: made where an element is encoded, or before (DrawsAhead::make), where a wavefront waits anyway:
// draw[c][k] = the draw of v[c][k], its upper 24 bits as a number.
struct DrawsInPlace {
    static constexpr bool kAhead = false;
};

// What the encoder needs to know about the elements a wavefront encodes.
struct EncodeRange {
    uint32_t len;         // valid elements
    uint64_t block;       // Philox block of the first one (a multiple of 16)
    uint32_t lane_block;  // Philox blocks from there to this lane's elements of chunk 0
    uint32_t row_groups;  // 64-element groups from row to row
    uint32_t k0, k1;      // Philox key
    uint32_t* words;      // the first element's packed words
};

template <int C>
struct DrawsAhead {
    static constexpr bool kAhead = true;
    float draw[C][4];
    // Chunks first + STRIDE c of the range into draw[c], c = BEGIN .. C - 1; LIMITED: those of them that begin below range.len.  (In the lean form: a
    // range that encode_is_plain() refuses has its draws made chunk by chunk.)
    template <class Layout, bool LIMITED, int STRIDE = 1, int BEGIN = 0>
    __device__ __forceinline__ void make(const EncodeRange& range, uint32_t first = 0)
    {
        if constexpr (BEGIN >= C) return;
        const PhiloxWords words = philox_words<(C - BEGIN > 4)>((uint32_t)(range.block >> 32), range.k0, range.k1);
#pragma unroll
        for (int c = BEGIN; c < C; ++c) {
            const uint32_t chunk = first + (uint32_t)(STRIDE * c);
            if (LIMITED && 256u * chunk >= range.len) continue;
            uint32_t r[4];
            philox4x32_10_uniform_c1((uint32_t)range.block + range.lane_block + Layout::kBlocks * chunk, words, r);
#pragma unroll
            for (int k = 0; k < 4; ++k) draw[c][k] = (float)(r[k] >> 8);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
};

// Levels up to which the rounding test takes its width already multiplied by 2^-24 (above, the width is a difference of
// two selected levels, see find_interval).
constexpr int kScaledWidthLevels = 4;
// Where the code is a sum of compares (LADDER in encode_chunks): three levels.  An element's code is the number of rungs k, 0 .. S - 2, with
// u * width_k < x - level_k: below its interval that never holds, as the right side is negative, and above it always, as x - level_k is then at
// least width_k, in fp32 too, and u * width_k at most the number below width_k.  That leaves intervals of width 0.  One that is not the last counts for
// every element from its level on: there the number below the level stands in its place.  The last one never counts.  No selects, and the products and
// compares of the rungs do not wait for each other: 25.6 M values in buckets of 32768, ORQ-3, 45.5 -> 44.3 us; with evenly spaced levels, whose
// two products are one and whose middle level is 0, TernGrad 21.8 -> 21.3.  Four levels take 14 instructions that way where the selects take
// 13, and were slower (44.0 -> 44.8).  Two levels have no selects to save (ORQ in buckets of 64 to 512 was 1 to 2 % slower; two elements side by side, which
// fill the wait, gained nothing); a single chunk does not earn back the numbers below the levels, which differ from lane to lane there (ORQ-3, 20 M values in
// buckets of 64: selects 48.8, sums 50.0).
template <int S, int C>
constexpr bool kLadder = S == 3 && C > 1;

// Index of an element's interval (see find_interval; five, eight or nine levels).
template <int S>
__device__ __forceinline__ uint32_t interval_index(float x, const float (&lv)[S])
{
    static_assert(S == 5 || S == 8 || S == 9, "two or three compares");
    if constexpr (S == 5) {
        const bool m1 = lv[2] <= x;
        const float t = m1 ? lv[3] : lv[1];
        return push_bit<true>(m1 ? 1u : 0u, __ballot(t <= x));
    } else {
        const bool m2 = lv[4] <= x;
        const float t1 = m2 ? lv[6] : lv[2];
        const bool m1 = t1 <= x;
        const float low7 = m2 ? (S == 9 ? lv[7] : __builtin_nanf("")) : lv[3];  // (the top level begins no interval)
        const float low5 = m2 ? lv[5] : lv[1];
        const float t0 = m1 ? low7 : low5;
        return push_bit<true>(push_bit<true>(m2 ? 1u : 0u, __ballot(m1)), __ballot(t0 <= x));
    }
}

// 4 x 4 transpose of the bits of every nibble position of four registers: bit p of nibble i of a[k] becomes bit k of nibble i of
// plane[p].
template <int BITS>
__device__ __forceinline__ void transpose_codes(const uint32_t (&a)[4], uint32_t (&plane)[BITS])
{
    auto select = [](uint32_t mask, uint32_t x, uint32_t y) __attribute__((always_inline)) { return (x & mask) | (y & ~mask); };
    uint32_t t[4];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        t[k] = select(0x33333333u, a[k], a[k + 2] << 2);
        t[k + 2] = select(0x33333333u, a[k] >> 2, a[k + 2]);
    }
#pragma unroll
    for (int p = 0; p < BITS; ++p)
        plane[p] = p % 2 == 0 ? select(0x55555555u, t[p & 2], t[(p & 2) + 1] << 1) : select(0x55555555u, t[p & 2] >> 1, t[(p & 2) + 1]);
}

// Encodes and packs chunks c0 .. c0 + GROUP - 1 (256 elements each).  CAREFUL: valid for every width and Philox block;
// otherwise encode_is_plain() holds.  EVEN: three levels -M, 0, M.  LADDER: see kLadder.
template <class Layout, int GROUP, int S, int BITS, Fill FILL, bool CAREFUL, bool AHEAD, bool EVEN, bool LADDER, class Pairs>
__device__ __forceinline__ void encode_chunks(const float (*v)[4], const float (&lv)[S], const float (&width)[S - 1], uint32_t c0,
                                              const EncodeRange& range, const PhiloxWords& words,
                                              const NibbleTranspose& transpose, uint32_t lane, Pairs pairs,
                                              const float (*ahead)[4] = nullptr)
{
    constexpr bool SCALED = !CAREFUL && S <= kScaledWidthLevels;
    static_assert(!LADDER || (S == 3 && !CAREFUL), "two rungs, finite widths");
    constexpr bool LOOKUP = !CAREFUL && Pairs::kUsed;
    constexpr int PLANES = 8 / GROUP;                // planes that share a register for the transpose
    constexpr int REGS = (BITS + PLANES - 1) / PLANES;
    const uint32_t len = range.len;
    uint32_t plane[BITS];
#pragma unroll
    for (int p = 0; p < BITS; ++p) plane[p] = 0;
    [[maybe_unused]] uint32_t code[4] = {0u, 0u, 0u, 0u};  // (LOOKUP) a nibble per chunk
    [[maybe_unused]] uint32_t rung[2] = {0u, 0u};          // (LADDER) a bit per element: past rung t
#pragma unroll
    for (int i = GROUP - 1; i >= 0; --i) {
        const uint32_t c = c0 + (uint32_t)i;
        if constexpr (FILL != Fill::kAll) {
            if (256u * c >= len) continue;
        }
        float draws[4];  // upper 24 bits
        [[maybe_unused]] uint32_t index[4];
        [[maybe_unused]] floatx2 level[4];
        if constexpr (LOOKUP) {  // the looks into LDS go ahead of the random numbers
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                index[k] = interval_index<S>(v[i][k], lv);
                level[k] = *(const LdsPair*)(uintptr_t)(pairs.table + 8u * index[k]);
            }
        }
        if constexpr (AHEAD) {
#pragma unroll
            for (int k = 0; k < 4; ++k) draws[k] = ahead[i][k];
        } else {
            uint32_t r[4];
            if constexpr (CAREFUL) {
                const uint64_t block = range.block + Layout::kBlocks * c + range.lane_block;
                philox4x32_10((uint32_t)block, (uint32_t)(block >> 32), range.k0, range.k1, r);
            } else {
                philox4x32_10_uniform_c1((uint32_t)range.block + range.lane_block + Layout::kBlocks * c, words, r);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) draws[k] = (float)(r[k] >> 8);
        }
#pragma unroll
        for (int k = 3; k >= 0; --k) {
            const float x = v[i][k];
            if constexpr (LOOKUP) {
                const bool up = draws[k] * level[k].y < x - level[k].x;
                code[k] = code[k] << 4 | (index[k] + (up ? 1u : 0u));
                continue;
            }
            if constexpr (LADDER) {
                push_less(rung[0], draws[k] * width[0], x - lv[0], rung[1], draws[k] * width[EVEN ? 0 : 1], EVEN ? x : x - lv[1]);
                continue;
            }
            const Interval<S> in = find_interval<S>(x, lv, width);
            const float delta = x - in.base;
            // u * width in fp32, u = the draw's upper 24 bits times 2^-24 (the factor is in the width where that is exact)
            const float draw = SCALED ? draws[k] : draws[k] * 0x1p-24f;
            const float scaled = draw * in.width;
            uint64_t carry = __ballot(scaled < delta);  // rounded up
#pragma unroll
            for (int p = 0; p < BITS; ++p) {
                const uint64_t index_bit = p < Interval<S>::kIndexBits ? in.bit[p < 3 ? p : 0] : 0ull;
                plane[p] = push_bit<S == 2>(plane[p], index_bit ^ carry);
                carry &= index_bit;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (LOOKUP) transpose_codes<BITS>(code, plane);
    if constexpr (LADDER) {
        plane[0] = rung[0] ^ rung[1];
        plane[BITS - 1] = rung[1];
    }
    if constexpr (GROUP == 1) {
        // a single chunk: the 8 lanes of a half word or their nibbles together, and lane p of them stores plane p
        const uint32_t j = lane & 7u, h = lane >> 3;
        uint32_t mine = 0;
#pragma unroll
        for (int p = 0; p < BITS; ++p) {
            uint32_t x = plane[p] << (4u * j);
            x |= dpp_u32<kDppXor1>(x);
            x |= dpp_u32<kDppXor2>(x);
            x |= dpp_u32<kDppHalfMirror>(x);
            mine = p == 0 || j == (uint32_t)p ? x : mine;
        }
        if (j < (uint32_t)BITS && (FILL != Fill::kRagged || 256u * c0 + 32u * h < ((len + 63u) & ~63u)))
            range.words[(Layout::group(c0, h, range.row_groups) * (uint32_t)BITS + j) * 2u + Layout::half(c0, h)] = mine;
        return;
    }
#pragma unroll
    for (int q = 0; q < REGS; ++q) {
        uint32_t x = plane[q * PLANES];
#pragma unroll
        for (int i = 1; i < PLANES; ++i)
            if (q * PLANES + i < BITS) x |= plane[q * PLANES + i < BITS ? q * PLANES + i : 0] << (4 * GROUP * i);
        x = nibble_transpose(x, transpose, lane);
        // lane 8 h + j now holds half word h (32 elements) of chunk c0 + j % GROUP of plane q * PLANES + j / GROUP
        const uint32_t j = lane & 7u, h = lane >> 3;
        const uint32_t c = c0 + (j & (uint32_t)(GROUP - 1)), p = (uint32_t)(q * PLANES) + j / (uint32_t)GROUP;
        const bool in_range = FILL == Fill::kAll || (FILL == Fill::kWholeChunks ? 256u * c < len
                                                                                : 256u * c + 32u * h < ((len + 63u) & ~63u));
        if ((BITS % PLANES == 0 || p < (uint32_t)BITS) && in_range)
            range.words[(Layout::group(c, h, range.row_groups) * (uint32_t)BITS + p) * 2u + Layout::half(c, h)] = x;
    }
}

// Whether the lean form of encode_chunks may be used: all of the range's Philox blocks share the upper counter word, and
// (where the widths are scaled) no width is so small that width * 2^-24 rounds.  Both hold for all but a few buckets
// that one meets in earnest.  The rungs of three levels also want finite widths.
template <int CHUNKS, int S, bool SCALED>
__device__ __forceinline__ bool encode_is_plain(const float (&width)[S - 1], const EncodeRange& range)
{
    bool plain = (uint32_t)range.block <= 0xFFFFFFFFu - 64u * CHUNKS;
    if constexpr (SCALED) {
        uint32_t smallest = 0xFFFFFFFFu;  // of the bit patterns minus 1: a width of 0 comes out largest
#pragma unroll
        for (int k = 0; k < S - 1; ++k) smallest = umin32(smallest, __float_as_uint(width[k]) - 1u);
        plain = plain && __ballot(smallest < __float_as_uint(0x1p-102f) - 1u) == 0;
    }
    if constexpr (kLadder<S, CHUNKS>) {
        bool finite = true;
#pragma unroll
        for (int k = 0; k < S - 1; ++k) finite = finite && __builtin_fabsf(width[k]) < __builtin_inff();
        plain = plain && __ballot(!finite) == 0;
    }
    return plain;
}

// v: the 256*C elements a wavefront holds (lane l, chunk c: elements 256c + 4l + {0..3} of the range that
// starts at global element `begin` and has `len` valid elements; FULL: len == 256*C); lv: the levels.
// reload(c, y) fetches the lane's four elements of chunk c once more.
//
// Bound by vector-instruction issue: Philox takes 9.5 instructions per element, the rounding test 5 or 6, the interval
// 0 .. 14 (find_interval).  The level index is assembled from the compare masks on the scalar unit, with three levels it is a sum of
// compares (kLadder).  Every bit plane keeps
// one register for up to 8 chunks: the elements are taken in descending order and each shifts its bit in (one
// instruction), so nibble c of lane l ends up holding the bits of this lane's four elements of chunk c.  One nibble
// transpose among 8 lanes then leaves 32 consecutive bits of a packed word in every lane, stored with one instruction
// for 8 chunks.  From five levels on, kernels with a grouped bucket in LDS keep the levels there once they are solved
// (PairsInLds): three or two compares give the interval's index, one look-up its level and width, and the index plus the carry is
// the code: 17.5 instead of 23 vector instructions per element beside Philox at eight levels (nine levels, buckets of 512, clipping,
// 25.6 M values 66.0 -> 63.3 us; eight levels, 32768 172.9 -> 167.1).  The rare range that encode_is_plain() refuses is encoded chunk by chunk in a loop.
template <class Layout, int C, int S, int BITS, Fill FILL, bool EVEN = false, bool VECTOR = false, class ReloadFn, class Pairs = NoPairs,
          class Draws = DrawsInPlace>
__device__ __forceinline__ void encode_all(const float (&v)[C][4], const float (&lv)[S], const EncodeRange& range, ReloadFn reload,
                                           Pairs pairs = Pairs{}, const Draws& draws = Draws{})
{
    constexpr bool SCALED = S <= kScaledWidthLevels || Pairs::kUsed;
    const uint32_t lane = threadIdx.x & 63u;
    float width[S - 1];
#pragma unroll
    for (int k = 0; k < S - 1; ++k) width[k] = lv[k + 1] - lv[k];
    const NibbleTranspose transpose = nibble_transpose_setup(lane);
    if (!encode_is_plain<C, S, SCALED>(width, range)) {
#pragma unroll 1
        for (uint32_t c = 0; 256u * c < range.len; ++c) {
            float y[1][4];
            reload(c, y[0]);
            encode_chunks<Layout, 1, S, BITS, FILL == Fill::kAll ? Fill::kRagged : FILL, true, false, EVEN, false>(y, lv, width, c, range, PhiloxWords{}, transpose, lane, NoPairs{});
        }
        return;
    }
    if constexpr (SCALED) {
#pragma unroll
        for (int k = 0; k < S - 1; ++k) width[k] *= 0x1p-24f;
    }
    float base[S];  // (see kLadder)
#pragma unroll
    for (int k = 0; k < S; ++k) base[k] = lv[k];
    if constexpr (kLadder<S, C>) {
#pragma unroll
        for (int k = 0; k < S - 1; ++k) {
            if (k < S - 2) base[k] = width[k] == 0.0f ? next_below(lv[k]) : lv[k];
            asm("" : "+v"(base[k]), "+v"(width[k]));
        }
    }
    if constexpr (Pairs::kUsed) {
        if (pairs.writer) {
#pragma unroll
            for (int k = 0; k < S - 1; ++k) ((LdsPair*)(uintptr_t)pairs.table)[k] = floatx2{lv[k], width[k]};
        }
        wave_lds_sync();
    }
    PhiloxWords words{};
    if constexpr (!Draws::kAhead) words = philox_words<VECTOR>((uint32_t)(range.block >> 32), range.k0, range.k1);
    constexpr int GROUP = C < 8 ? C : 8;
#pragma unroll
    for (int c0 = C - GROUP; c0 >= 0; c0 -= GROUP) {
        if constexpr (FILL != Fill::kAll) {
            if (256u * (uint32_t)c0 >= range.len) continue;  // nothing in these chunks: no words to write
        }
        const float(*ahead)[4] = nullptr;
        if constexpr (Draws::kAhead) ahead = &draws.draw[c0];
        encode_chunks<Layout, GROUP, S, BITS, FILL, false, Draws::kAhead, EVEN, kLadder<S, C>>(&v[c0], base, width, (uint32_t)c0, range, words, transpose, lane, pairs, ahead);
    }
}

// The `len` elements from global element `begin` on, as orq_encode takes them.
template <int BITS>
__device__ __forceinline__ EncodeRange one_range(uint32_t len, size_t begin, uint64_t seed, uint64_t index_offset, uint32_t* codes32)
{
    return EncodeRange{uniform_u32(len), (index_offset + begin) >> 2, threadIdx.x & 63u, 1u, (uint32_t)seed, (uint32_t)(seed >> 32),
                       codes32 + begin / 64 * (2 * BITS)};
}

template <int C, int S, int BITS, bool FULL, bool EVEN = false, bool VECTOR = false, class ReloadFn, class Pairs = NoPairs, class Draws = DrawsInPlace>
__device__ __forceinline__ void orq_encode(const float (&v)[C][4], const float (&lv)[S], uint32_t len, size_t begin,
                                           uint64_t seed, uint64_t index_offset, uint32_t* __restrict__ codes32, ReloadFn reload,
                                           Pairs pairs = Pairs{}, const Draws& draws = Draws{})
{
    encode_all<OneRange, C, S, BITS, FULL ? Fill::kAll : Fill::kRagged, EVEN, VECTOR>(v, lv, one_range<BITS>(len, begin, seed, index_offset, codes32), reload,
                                                                        pairs, draws);
}

// The table of levels of wavefront `wave` in the place of a grouped bucket, once the levels are solved (five and more of them).
template <int S, bool GROUPED>
__device__ __forceinline__ auto encoder_table(uint32_t* grouped, uint32_t wave)
{
    if constexpr (GROUPED && S > kScaledWidthLevels)
        return PairsInLds{(uint32_t)(uintptr_t)((LdsWord*)grouped) + 64u * wave, (threadIdx.x & 63u) == 0u};
    else
        return NoPairs{};
}

// The elements [first, first + my_len) of the bucket of `len` elements at g, read once (past the caches), element
// 256 c + 4 lane + k of the range into v[c][k]; padding holds PAD.  A range shorter than its capacity takes whole 16-byte
// loads too: the lanes past its end read the bucket's first elements and drop them, and where its length is not a
// multiple of 4 (a ragged last bucket) the quad it ends in is filled from three loads of the whole wavefront.
template <int C, bool FULL>
__device__ __forceinline__ void load_range(float (&v)[C][4], const float* __restrict__ g, uint32_t first, uint32_t len,
                                           uint32_t my_len, uint32_t lane, float pad = kNoElement)
{
    float tail[3] = {pad, pad, pad};
    const uint32_t quad = my_len / 4u;
    if constexpr (!FULL) {
        if (my_len % 4u != 0u) {
            const float* t = g + first + 4u * quad;
            tail[0] = t[0];
            if (my_len % 4u > 1u) tail[1] = t[1];
            if (my_len % 4u > 2u) tail[2] = t[2];
        }
    }
    if (FULL || len >= 4u) {
        floatx4 q[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const uint32_t e = 256u * c + 4u * lane;
            const bool inside = FULL || e + 4u <= my_len;
            q[c] = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(g + (inside ? first + e : 0u)));
        }
        // All loads ahead of the first use: where registers are few the compiler waits for half of them before it makes the other half's addresses, a
        // second trip to memory (20 M values in buckets of 5120: five evenly spaced levels 29.7 -> 28.4 us, Linear-5 45.8 -> 44.4).  Scalar and LDS
        // instructions may pass.  (One or two loads are not split, and lose 0.1 us.)
        if constexpr (!FULL && C >= 4) __builtin_amdgcn_sched_barrier(0x84);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const bool inside = FULL || 256u * c + 4u * lane + 4u <= my_len;
            v[c][0] = inside ? q[c].x : pad; v[c][1] = inside ? q[c].y : pad;
            v[c][2] = inside ? q[c].z : pad; v[c][3] = inside ? q[c].w : pad;
        }
    } else {
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) v[c][k] = pad;
    }
    if constexpr (!FULL) {
        if (my_len % 4u != 0u) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const bool mine = 64u * c + lane == quad;
#pragma unroll
                for (int k = 0; k < 3; ++k) v[c][k] = mine ? tail[k] : v[c][k];
            }
        }
    }
}

// Padding of a wavefront's elements: fminf and fmaxf pass over it, no comparison with it holds.
template <int C>
__device__ __forceinline__ void set_padding(float (&v)[C][4], uint32_t my_len, uint32_t lane)
{
    asm volatile("" : "+v"(lane));  // tested afresh: the lane masks of an earlier pass would not fit the scalar registers
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[c][k] = 256u * c + 4u * lane + k < my_len ? v[c][k] : kNoElement;
}

// Smallest and largest element that the lane holds, and (ZEROS) how many zeros; padding is NaN.
template <int C, bool ZEROS>
__device__ __forceinline__ void lane_extremes(const float (&v)[C][4], float& low, float& high, uint32_t& zeros)
{
    low = __uint_as_float(0x7F800000u);
    high = __uint_as_float(0xFF800000u);
    zeros = 0u;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            low = fminf(low, v[c][k]);
            high = fmaxf(high, v[c][k]);
            if constexpr (ZEROS) zeros += v[c][k] == 0.0f ? 1u : 0u;
        }
}

// Counts the lane's elements into their bins; slot = bin | position inside the bin << 16 (pack_slot).  The returning LDS
// add hands every element its position.  No answer is waited for before the last add of a group has been sent, and the
// elements of the chunk that the range ends in take no branch: padding adds 0 to one bin per lane.
template <int C, bool FULL, int HALF, int SHIFT>
__device__ __forceinline__ void count_into_bins(uint32_t (&slot)[C][4], const float (&v)[C][4], uint32_t* bins, uint32_t t_low,
                                                uint32_t my_len, uint32_t lane)
{
    // (a range that does not fill its registers: in groups of four chunks, for the sake of the register count)
    constexpr int GROUP = FULL || C < 4 ? C : 4;
    const float zero = opaque_zero();
    if constexpr (!FULL) asm volatile("" : "+v"(lane));  // (see set_padding)
#pragma unroll
    for (int c0 = 0; c0 < C; c0 += GROUP) {
        uint32_t position[GROUP][4];
#pragma unroll
        for (int i = 0; i < GROUP; ++i) {
            const int c = c0 + i;
            if (FULL || 256u * (uint32_t)(c + 1) <= my_len) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    slot[c][k] = value_bin<HALF, SHIFT>(v[c][k] + zero, t_low);
                    position[i][k] = atomicAdd(&bins[slot[c][k]], 1u);
                }
            } else if (256u * (uint32_t)c < my_len) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const bool valid = 256u * c + 4u * lane + k < my_len;
                    slot[c][k] = valid ? value_bin<HALF, SHIFT>(v[c][k] + zero, t_low) : lane;
                    position[i][k] = atomicAdd(&bins[slot[c][k]], valid ? 1u : 0u);
                }
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) slot[c][k] = position[i][k] = 0u;
            }
        }
#pragma unroll
        for (int i = 0; i < GROUP; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) slot[c0 + i][k] = pack_slot(position[i][k], slot[c0 + i][k], (uint32_t)HALF);
    }
}

// Scatters the lane's elements into their bins.  The bin starts of a group of elements are all read before the group's
// values are written (a read behind a write to the same LDS object would wait for it).  Padding of a group that holds
// elements goes where it lies in the bucket, behind all elements, as zeros.
template <int C, bool FULL>
__device__ __forceinline__ void scatter_into_bins(uint32_t* grouped, const uint32_t* bin_start_middle, const uint32_t (&slot)[C][4],
                                                  const float (&v)[C][4], uint32_t first, uint32_t my_len, uint32_t lane)
{
    constexpr int GROUP = C < 4 ? C : 4;
    if constexpr (!FULL) asm volatile("" : "+v"(lane));  // (see set_padding)
    auto scatter_group = [&](int c0, auto all) __attribute__((always_inline)) {
        uint32_t to[GROUP][4];
#pragma unroll
        for (int c = 0; c < GROUP; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                to[c][k] = slot_bin_start(bin_start_middle, slot[c0 + c][k]) + (slot[c0 + c][k] >> 16);
#pragma unroll
        for (int c = 0; c < GROUP; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if constexpr (!decltype(all)::value) {
                    const uint32_t e = 256u * (uint32_t)(c0 + c) + 4u * lane + k;
                    to[c][k] = e < my_len ? to[c][k] : first + e;
                }
                uint32_t bits = __float_as_uint(v[c0 + c][k]);
                if constexpr (!decltype(all)::value) bits = 256u * (uint32_t)(c0 + c) + 4u * lane + k < my_len ? bits : 0u;
                grouped[to[c][k]] = bits;
            }
    };
#pragma unroll
    for (int c0 = 0; c0 < C; c0 += GROUP) {
        if (FULL || 256u * (uint32_t)(c0 + GROUP) <= my_len) scatter_group(c0, std::true_type{});
        else if (256u * (uint32_t)c0 < my_len) scatter_group(c0, std::false_type{});
    }
}

// fp64 sum of the 4 C grouped positions of thread `thread`; the bucket has `len` of them, zeros behind them up to the end of the
// thread's positions, if those begin below `len`.  16-byte reads; every thread begins at another of its pieces, so that
// neighbours meet different LDS banks.
template <int C>
__device__ __forceinline__ double sum_of_positions(const uint32_t* grouped, uint32_t thread, uint32_t len)
{
    const float4* from = reinterpret_cast<const float4*>(grouped) + C * thread;
    const uint32_t turn = thread / (C < 8 ? 8u / C : 1u);
    double part = 0.0;
#pragma unroll
    for (uint32_t q = 0; q < (uint32_t)C; ++q) {
        const float4 x = from[(q + turn) & (uint32_t)(C - 1)];
        part += (double)x.x;
        part += (double)x.y;
        part += (double)x.z;
        part += (double)x.w;
    }
    return 4u * C * thread < len ? part : 0.0;
}

// The reload function of orq_encode for a range in memory: g = its first element; limit = the clipping threshold
// (infinity: none).
struct ReloadFromMemory {
    const float* g;
    uint32_t len;
    float limit;
    __device__ __forceinline__ void operator()(uint32_t c, float (&y)[4]) const
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t e = 256u * c + 4u * (threadIdx.x & 63u) + (uint32_t)k;
            y[k] = e < len ? clipped(g[e], limit) : kNoElement;
        }
    }
};

// Whether the bucket holds a non-zero element more than safe_binades(capacity) binades below its largest magnitude
// (mag_max = its bit pattern), i.e. whether its fp64 sums may round.  Such elements sit in the bins next to zero: the
// two centre bins, which take everything below the binned range, and above 4096 elements also the lowest regular bins.
// Called by `threads` threads (thread = 0 .. threads - 1) once the bucket is grouped; every thread looks at its share
// of those bins and returns what it saw: the caller combines the answers.
template <int HALF, int SHIFT, class Lds>
__device__ __forceinline__ bool any_tiny_element(const Lds& lds, uint32_t capacity, uint32_t mag_max, uint32_t t_low,
                                                 uint32_t thread, uint32_t threads)
{
    const uint32_t safe = safe_binades(capacity);
    const uint32_t biased = mag_max >> 23;
    if (biased <= safe) return false;  // every element is a multiple of 2^-149 and the sums stay below 2^53 of those
    const uint32_t mag_safe = (biased - safe) << 23;  // bit pattern of the smallest safe magnitude
    const uint32_t t_safe = mag_safe >> SHIFT;
    uint32_t bins = t_safe > t_low ? t_safe - t_low : 1u;  // bins per sign that may hold smaller elements
    bins = bins > (uint32_t)HALF ? (uint32_t)HALF : bins;
    const uint32_t first = uniform_u32(lds.bin_start[(uint32_t)HALF - bins]);
    const uint32_t last = uniform_u32(lds.bin_start[(uint32_t)HALF + bins]);
    bool tiny = false;
    for (uint32_t i = first + thread; i < last; i += threads) {
        const uint32_t magnitude = lds.grouped[i] & 0x7FFFFFFFu;
        tiny = tiny || (magnitude != 0u && magnitude < mag_safe);
    }
    return tiny;
}

// Where the levels come from; all rules share the random-rounding encoder.
//   kOptimal: ORQ (Theorem 1, Algorithm 1).
//   kPb: BinGrad-pb (Section 3.2): two levels -b_1, +b_1 from the scheme's optimal condition instead of the
//        bucket extremes; the encoder then clamps everything outside them.
//   kEven: QSGD-s / TernGrad (Section 3.1): S levels evenly spaced from -M to +M, M the largest magnitude.
//   kLinear: Linear-s (Section 5): the order statistics at the fractions k/(S-1) of the sorted bucket.
enum LevelRule { kOptimal = 0, kPb = 1, kEven = 2, kLinear = 3 };

// Lane `at` (wave-uniform) of a 64-bit value.
__device__ __forceinline__ double lane_entry_f64(double x, uint32_t at)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, at), hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), at);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// One level solve (discrete optimal condition, second remark after Theorem 1): level k between the current
// levels l and r, whose records (and k's) are in lds.lvl_*.  Run by one whole wavefront.
template <class Lds, class PickFn>
__device__ __forceinline__ void orq_solve_one(Lds& lds, PickFn pick, uint32_t k, uint32_t l, uint32_t r, uint32_t len,
                                              double bound, uint32_t lane)
{
    const float L = uniform_f32(lds.lvl_value[l]);
    const float R = uniform_f32(lds.lvl_value[r]);
    const uint32_t cnt_lt_L = uniform_u32(lds.lvl_count_lt[l]);
    const uint32_t cnt_le_R = uniform_u32(lds.lvl_count_le[r]);
    const double sum_lt_L = uniform_f64(lds.lvl_sum_lt[l]);
    const double sum_le_R = uniform_f64(lds.lvl_sum_le[r]);
    const uint32_t last_rank = uniform_u32(lds.lvl_rank[k]);  // read with the others: one wait for all of them
    bool copy_left = !(L < R);
    Picked p;
    uint32_t rank = 0;
    if (!copy_left) {
        // S = sum_{L<=v<=R} (v - L),  T = S / (R - L),  level = element of rank #{v<=R} - floor(T)
        const uint32_t count_in = cnt_le_R - cnt_lt_L;
        const double Ssum = (sum_le_R - sum_lt_L) - (double)L * (double)count_in;
        const double width = (double)R - (double)L;
        double m;
        if (!floor_t_from_sums(Ssum, width, bound, m)) {
            // the fp64 sums do not decide floor(T): exact sums of the elements in [L, R] (rare)
            m = (double)exact_floor_t_grouped(
                lds.exact_limb[(threadIdx.x >> 6) & (sizeof(lds.exact_limb) / sizeof(lds.exact_limb[0]) - 1u)], lds.grouped, len,
                lane, kWave, L, R, count_in, (uint32_t)m);
        }
        // rank = cnt_le_R - m, at least 1 and at most len
        const uint32_t below = uniform_u32((uint32_t)m);
        rank = below >= cnt_le_R ? 1u : cnt_le_R - below;
        rank = rank > len ? len : rank;
        if (rank == last_rank) return;  // same element as last time
        p = pick(rank);
        if (key_to_float(p.key) < L) copy_left = true;
    }
    __builtin_amdgcn_wave_barrier();
    if (lane == 0u) {
        if (copy_left) {
            // the level coincides with the left end (L == R, or rounding put it below L)
            lds.lvl_value[k] = L;
            lds.lvl_count_lt[k] = cnt_lt_L;
            lds.lvl_sum_lt[k] = sum_lt_L;
            lds.lvl_count_le[k] = (L < R) ? uniform_u32(lds.lvl_count_le[l]) : cnt_le_R;
            lds.lvl_sum_le[k] = (L < R) ? uniform_f64(lds.lvl_sum_le[l]) : sum_le_R;
            lds.lvl_rank[k] = 0u;
        } else {
            lds.lvl_value[k] = key_to_float(p.key);
            lds.lvl_count_lt[k] = p.count_lt;
            lds.lvl_count_le[k] = p.count_le;
            lds.lvl_sum_lt[k] = p.sum_lt;
            lds.lvl_sum_le[k] = p.sum_le;
            lds.lvl_rank[k] = rank;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The level records of a bucket held by the wavefront itself (wave-uniform values in registers): what lds.lvl_* keeps,
// for the kernels whose solves all have compile-time level indices.
template <int S>
struct LevelRecords {
    float value[S];
    uint32_t count_lt[S], count_le[S], rank[S];
    double sum_lt[S], sum_le[S];
};

// orq_solve_one on such records: level K between the levels L_ and R_.
template <int K, int L_, int R_, int S, class Lds, class PickFn>
__device__ __forceinline__ void orq_solve_one_in_registers(LevelRecords<S>& st, Lds& lds, PickFn pick, uint32_t len,
                                                           double bound, uint32_t lane)
{
    const float L = st.value[L_], R = st.value[R_];
    const uint32_t cnt_lt_L = st.count_lt[L_], cnt_le_R = st.count_le[R_];
    const double sum_lt_L = st.sum_lt[L_], sum_le_R = st.sum_le[R_];
    if (!(L < R)) {
        // the level coincides with both ends
        st.value[K] = L;
        st.count_lt[K] = cnt_lt_L;
        st.sum_lt[K] = sum_lt_L;
        st.count_le[K] = cnt_le_R;
        st.sum_le[K] = sum_le_R;
        st.rank[K] = 0u;
        return;
    }
    // S = sum_{L<=v<=R} (v - L),  T = S / (R - L),  level = element of rank #{v<=R} - floor(T)
    const uint32_t count_in = cnt_le_R - cnt_lt_L;
    const double Ssum = (sum_le_R - sum_lt_L) - (double)L * (double)count_in;
    const double width = (double)R - (double)L;
    double m;
    if (!floor_t_from_sums(Ssum, width, bound, m)) {
        // the fp64 sums do not decide floor(T): exact sums of the elements in [L, R] (rare)
        m = (double)exact_floor_t_grouped(lds.exact_limb[0], lds.grouped, len, lane, kWave, L, R, count_in, (uint32_t)m);
    }
    // rank = cnt_le_R - m, at least 1 and at most len
    const uint32_t below = uniform_u32((uint32_t)m);
    uint32_t rank = below >= cnt_le_R ? 1u : cnt_le_R - below;
    rank = rank > len ? len : rank;
    if (rank == st.rank[K]) return;  // same element as last time
    const Picked p = pick(rank);
    if (key_to_float(p.key) < L) {
        // rounding put the level below L: it coincides with the left end
        st.value[K] = L;
        st.count_lt[K] = cnt_lt_L;
        st.sum_lt[K] = sum_lt_L;
        st.count_le[K] = st.count_le[L_];
        st.sum_le[K] = st.sum_le[L_];
        st.rank[K] = 0u;
    } else {
        st.value[K] = key_to_float(p.key);
        st.count_lt[K] = p.count_lt;
        st.count_le[K] = p.count_le;
        st.sum_lt[K] = p.sum_lt;
        st.sum_le[K] = p.sum_le;
        st.rank[K] = rank;
    }
}

// Schedule of the level solves over the first two wavefronts of a team (Algorithm 1 and the re-solve sweeps;
// the results are those of the serial order).  Greedy: after the root, the solves of the left half only touch levels
// up to the root and those of the right half only levels from the root on, so wavefront 0 takes the left and
// wavefront 1 the right half, step by step.  Sweeps, two at a time: wavefront 0 runs sweep s, wavefront 1 sweep
// s + 1 two levels behind it (level k of a sweep needs level k - 1 of the same sweep and level k + 1 of the sweep
// before).  Where wavefront 0 runs out of greedy solves before wavefront 1 (8 levels), it starts the first sweep in
// those steps.  Every wavefront of the workgroup must call this; a workgroup barrier ends every step.
struct TeamGreedy {
    uint16_t entry[2][8];  // k | l << 4 | r << 8 per wavefront and step; 0 = idle
    int steps;
    // Greedy steps in which wavefront 0 has nothing left to do and can already run the first solves of the first
    // sweep (levels 1, 2): head_step[h] = the step that takes level h + 1, or -1.  Possible when the greedy value of
    // level h + 2 is final by then and the solve of wavefront 1 in that step touches none of the levels h .. h + 2.
    int head_step[2];
    int head;
};

template <int S>
constexpr TeamGreedy team_greedy()
{
    const GreedyOrder o = greedy_order<S>();
    TeamGreedy g{{{0, 0, 0, 0, 0, 0, 0, 0}, {0, 0, 0, 0, 0, 0, 0, 0}}, 0, {-1, -1}, 0};
    int next[2] = {1, 1};
    int root = 0;
    for (int i = 0; i < o.count; ++i) {
        const uint32_t e = (uint32_t)(o.packed[i / 5] >> (12 * (i % 5))) & 0xFFFu;
        const int k = (int)(e & 15u);
        if (i == 0) {
            root = k;
            g.entry[0][0] = (uint16_t)e;
        } else {
            const int w = k < root ? 0 : 1;
            g.entry[w][next[w]++] = (uint16_t)e;
        }
    }
    g.steps = o.count == 0 ? 0 : (next[0] > next[1] ? next[0] : next[1]);
    g.head_step[0] = g.head_step[1] = -1;
    g.head = 0;
    for (int step = 1; step < g.steps && g.head < 2; ++step) {
        if (g.entry[0][step] != 0) continue;
        bool later_work = false;  // only trailing idle steps of wavefront 0
        for (int q = step; q < g.steps; ++q) later_work = later_work || g.entry[0][q] != 0;
        if (later_work) continue;
        const int h = g.head, level = h + 1;
        if (level > S - 2) break;
        // greedy value of level + 1 final before this step (or it is the top level)
        bool right_final = level + 1 == S - 1;
        for (int w = 0; w < 2; ++w)
            for (int q = 0; q < step; ++q)
                if (g.entry[w][q] != 0 && (int)(g.entry[w][q] & 15u) == level + 1) right_final = true;
        const uint32_t other = g.entry[1][step];
        const int ok = (int)(other & 15u), ol = (int)((other >> 4) & 15u), orr = (int)((other >> 8) & 15u);
        const bool apart = other == 0 || ((ok < level - 1 || ok > level + 1) && ol != level && orr != level);
        if (!right_final || !apart) break;
        g.head_step[h] = step;
        ++g.head;
    }
    return g;
}

// The greedy steps are unrolled (their level indices are compile-time constants: measured 3-4 % faster on 8 levels
// than one loop over a packed table, at equal register counts).
template <int S, class Lds, class PickFn>
__device__ __forceinline__ void orq_team_solve(Lds& lds, PickFn pick, uint32_t wave, uint32_t len, uint32_t sweeps,
                                               uint32_t lane)
{
    constexpr TeamGreedy greedy = team_greedy<S>();
    constexpr uint32_t INTERIOR = S - 2;
    const double bound = uniform_f64(lds.sum_error_bound);  // (see floor_t_from_sums)
#pragma unroll
    for (int step = 0; step < greedy.steps; ++step) {
        if (wave < 2u) {
            const uint32_t e = wave == 0u ? greedy.entry[0][step] : greedy.entry[1][step];
            if (e != 0u) orq_solve_one(lds, pick, e & 15u, (e >> 4) & 15u, (e >> 8) & 15u, len, bound, lane);
            if (wave == 0u && sweeps > 0u) {  // head start of the first sweep
                if (greedy.head_step[0] == step) orq_solve_one(lds, pick, 1u, 0u, 2u, len, bound, lane);
                if (greedy.head_step[1] == step) orq_solve_one(lds, pick, 2u, 1u, 3u, len, bound, lane);
            }
        }
        __syncthreads();
    }
    for (uint32_t s = 0; s < sweeps; s += 2u) {
        const bool pair = s + 1u < sweeps;
        const uint32_t steps = INTERIOR + (pair ? 2u : 0u);
        for (uint32_t t = (s == 0u ? (uint32_t)greedy.head : 0u); t < steps; ++t) {
            if (wave == 0u && t < INTERIOR) orq_solve_one(lds, pick, t + 1u, t, t + 2u, len, bound, lane);
            if (wave == 1u && pair && t >= 2u) orq_solve_one(lds, pick, t - 1u, t - 2u, t, len, bound, lane);
            __syncthreads();
        }
    }
}

// fp64 sum of the grouped positions [0, position), position < bucket length: the prefix of its block plus the
// block's positions before it.
template <class Lds>
__device__ __forceinline__ double sum_before_position(const Lds& lds, uint32_t position, uint32_t lane)
{
    constexpr uint32_t BLOCK = Lds::BLOCK;
    const uint32_t block = position / BLOCK;
    const uint32_t block_first = block * BLOCK;
    const float head = lane < position - block_first ? __uint_as_float(lds.grouped[block_first + lane]) : 0.0f;
    return uniform_f64(lds.block_prefix[block]) + wave_sum((double)head);
}

// Run solve(k, l, r) with compile-time level indices: the greedy order of Algorithm 1, and one re-solve sweep.
template <int S, int STEP, class Solve>
__device__ __forceinline__ void for_greedy_steps(Solve&& solve)
{
    constexpr GreedyOrder order = greedy_order<S>();
    if constexpr (STEP < order.count) {
        constexpr uint32_t e =
            STEP < 5 ? (uint32_t)(order.packed[0] >> (12 * STEP)) : (uint32_t)(order.packed[1] >> (12 * (STEP - 5)));
        solve(std::integral_constant<int, (int)(e & 15u)>{}, std::integral_constant<int, (int)((e >> 4) & 15u)>{},
              std::integral_constant<int, (int)((e >> 8) & 15u)>{});
        for_greedy_steps<S, STEP + 1>(solve);
    }
}

template <int S, int K, class Solve>
__device__ __forceinline__ void for_sweep_levels(Solve&& solve)
{
    if constexpr (K + 1 < S) {
        solve(std::integral_constant<int, K>{}, std::integral_constant<int, K - 1>{}, std::integral_constant<int, K + 1>{});
        for_sweep_levels<S, K + 1>(solve);
    }
}

// The level solves of one bucket, run by one wavefront once the bucket is grouped in LDS and the level
// records of the two ends are set.  pick(rank) returns the element of that 1-based rank (Picked); `zeros` is the
// number of zeros in the bucket (BinGrad-pb only).  Interior levels end up in lds.lvl_value; returns b_1 for
// BinGrad-pb.
template <int S, int RULE, class Lds, class PickFn, class EdgeFn>
__device__ __forceinline__ float orq_solve_levels(Lds& lds, PickFn pick, EdgeFn lower_edge_of_bin, uint32_t len,
                                                  uint32_t zeros, uint32_t sweeps, uint32_t lane)
{
    constexpr bool PB = RULE == kPb;
    float pb_level = 0.0f;
    if constexpr (PB) {
        // ---- b_1: minimise |b * #{v > 0} - sum_{v >= b} v| over the positive bucket values.  The
        //      difference grows with b, so the minimiser is one of the two values around its sign
        //      change, which a bisection over the ranks of the positive values finds. -------------
                const uint32_t not_positive = uniform_u32(lds.bin_start[Lds::B / 2]) + zeros;  // negatives fill the lower bins
        const uint32_t positives = len - not_positive;
        const double total = uniform_f64(lds.lvl_sum_le[S - 1]);
        if (positives > 0u) {
            // First the bin: every element of a positive bin j lies below the lower edge e of bin j + 1, so its
            // gap is below gap(e) = e * #{v > 0} - (sum of the bins above j); the wanted value sits in the first bin
            // j whose gap(e) is not negative, or is the first element after it.  One block-prefix look-up per step.
            uint32_t bin_lo = (uint32_t)(Lds::B / 2), bin_hi = (uint32_t)Lds::B - 1u;
            // All positive bins at once, one per lane: the sum before a position lies between the prefixes of the
            // block it falls into and of the next block (positive bins hold positive values), which brackets
            // gap(e) from both sides and decides its sign for every bin except the few whose first position shares
            // a block with the sign change; the bisection then runs over those only.  (A block that begins among the
            // negative values gives no lower bracket.)
            const uint32_t first_not_negative = uniform_u32(lds.bin_start[Lds::B / 2]);
            for (uint32_t bin0 = (uint32_t)(Lds::B / 2); bin0 < (uint32_t)Lds::B; bin0 += kWave) {
                const uint32_t bin = bin0 + lane;
                const uint32_t above = lds.bin_start[bin + 1u];
                const uint32_t block = above / (uint32_t)Lds::BLOCK;
                const bool inside = above < len;  // otherwise nothing lies above the bin: gap(e) >= 0
                const double before_lo = inside ? lds.block_prefix[block] : total;
                const double before_hi =
                    inside && (block + 1u) * (uint32_t)Lds::BLOCK < len ? lds.block_prefix[block + 1u] : total;
                const double scaled_edge = (double)lower_edge_of_bin(bin + 1u) * (double)positives;
                const bool bracketed_below = !inside || block * (uint32_t)Lds::BLOCK >= first_not_negative;
                const uint64_t surely_not_negative =
                    __ballot(bracketed_below && scaled_edge - (total - before_lo) >= 0.0);
                const uint64_t surely_negative = __ballot(scaled_edge - (total - before_hi) < 0.0);
                if (surely_negative != 0)
                    bin_lo = umax32(bin_lo, bin0 + 64u - (uint32_t)__builtin_clzll(surely_negative));
                if (surely_not_negative != 0)
                    bin_hi = umin32(bin_hi, bin0 + (uint32_t)__builtin_ctzll(surely_not_negative));
            }
            if (bin_lo > bin_hi) bin_lo = bin_hi;  // only rounding can make the two bounds cross
            while (bin_lo < bin_hi) {
                const uint32_t mid = (bin_lo + bin_hi) >> 1;
                const uint32_t above = uniform_u32(lds.bin_start[mid + 1u]);  // first position of the bins above mid
                const double sum_above = above < len ? total - sum_before_position(lds, above, lane) : 0.0;
                const double gap = (double)lower_edge_of_bin(mid + 1u) * (double)positives - sum_above;
                if (gap >= 0.0) bin_hi = mid;
                else bin_lo = mid + 1u;
            }
            const uint32_t first_of_bin = uniform_u32(lds.bin_start[bin_lo]);
            const uint32_t first_above = uniform_u32(lds.bin_start[bin_lo + 1u]);
            // Then the value inside it.  A bin of at most 64 elements is sorted once and every distinct positive value
            // of it gets its gap in its own lane (the sum of the strictly smaller elements is an exclusive scan at the
            // first lane that holds the value); where none of them is the wanted one, that is the first element above the bin.
            const uint32_t count = first_above - first_of_bin;
            bool done = false;
            if (count > 0u && count <= 64u) {
                const uint32_t mine = lane < count ? stored_key(lds.grouped[first_of_bin + lane]) : 0xFFFFFFFFu;
                const uint32_t sorted = wave_sort_u32(mine, lane, count);
                const float value = lane < count ? key_to_float(sorted) : 0.0f;
                const double below_bin = sum_before_position(lds, first_of_bin, lane);
                const double smaller = below_bin + (wave_inclusive_scan_f64((double)value) - (double)value);
                const uint32_t previous = (uint32_t)__shfl_up((int)sorted, 1, kWave);
                const bool candidate = lane < count && value > 0.0f && (lane == 0u || previous != sorted);
                const double gap = (double)value * (double)positives - (total - smaller);
                const uint64_t not_negative = __ballot(candidate && gap >= 0.0);
                if (not_negative != 0 || first_above < len) {
                    // first lane of the wanted value; past the bin's: it is the first element above the bin
                    const uint32_t at = not_negative != 0 ? (uint32_t)__builtin_ctzll(not_negative) : count;
                    double gap_up;
                    if (not_negative != 0) {
                        pb_level = key_to_float(__builtin_amdgcn_readlane(sorted, at));
                        gap_up = lane_entry_f64(gap, at);
                    } else {
                        const Picked up = pick(first_above + 1u);
                        pb_level = key_to_float(up.key);
                        gap_up = (double)pb_level * (double)positives - (total - up.sum_lt);
                    }
                    const uint32_t count_lt = first_of_bin + at;  // elements of the bucket below the wanted value
                    if (count_lt > not_positive) {  // a smaller positive value exists
                        float down;
                        double gap_down;
                        if (at > 0u) {
                            const uint32_t down_key = __builtin_amdgcn_readlane(sorted, at - 1u);
                            const uint32_t down_at = (uint32_t)__popcll(__ballot(sorted < down_key));  // its first lane
                            down = key_to_float(down_key);
                            gap_down = lane_entry_f64(gap, down_at);
                        } else {
                            const Picked below = pick(count_lt);
                            down = key_to_float(below.key);
                            gap_down = (double)down * (double)positives - (total - below.sum_lt);
                        }
                        if (fabs(gap_down) <= fabs(gap_up)) pb_level = down;  // ties take the smaller value
                    }
                    done = true;
                }
            }
            if (!done) {
                // A crowded bin, an empty one, or the last one that holds elements.  The gap grows with the value also between the
                // bin's elements: a bisection over the keys finds the smallest one whose gap is not negative, each step one sum
                // over the bin, and the wanted value is the first element from there on.
                auto each = [&](auto f) __attribute__((always_inline)) {
#pragma unroll 1
                    for (uint32_t i = lane; i < count; i += kWave) f(__uint_as_float(lds.grouped[first_of_bin + i]) + 0.0f);
                };
                const double below_bin = count != 0u ? sum_before_position(lds, first_of_bin, lane) : 0.0;
                auto smaller_than = [&](float t) __attribute__((always_inline)) {  // sum of the bucket's elements below t, t in the bin
                    double part = 0.0;
                    each([&](float x) __attribute__((always_inline)) { part += (double)(x < t ? x : 0.0f); });
                    return below_bin + wave_sum(part);
                };
                uint32_t lo = 0xFFFFFFFFu, largest = 0u;  // keys of the bin's positive elements
                each([&](float x) __attribute__((always_inline)) {
                    lo = x > 0.0f ? umin32(lo, float_to_key(x)) : lo;
                    largest = x > 0.0f ? umax32(largest, float_to_key(x)) : largest;
                });
                lo = wave_min_u32(lo);
                largest = wave_max_u32(largest);
                uint32_t hi = largest + 1u;  // (no positive element: 1, and lo lies above)
                while (lo < hi) {
                    const uint32_t mid = lo + ((hi - lo) >> 1);
                    const float t = key_to_float(mid);
                    if ((double)t * (double)positives - (total - smaller_than(t)) >= 0.0) hi = mid;
                    else lo = mid + 1u;
                }
                // the first element from `lo` on: in the bin, or above it; the bucket's last where only rounding (or NaN) says that there is none
                double gap_up;
                uint32_t count_lt = 0;  // elements of the bucket below it
                if (lo <= largest) {
                    uint32_t up = 0xFFFFFFFFu;
                    each([&](float x) __attribute__((always_inline)) { up = float_to_key(x) >= lo ? umin32(up, float_to_key(x)) : up; });
                    pb_level = key_to_float(wave_min_u32(up));
                    gap_up = (double)pb_level * (double)positives - (total - smaller_than(pb_level));
                    each([&](float x) __attribute__((always_inline)) { count_lt += x < pb_level ? 1u : 0u; });
                    count_lt = first_of_bin + wave_sum_u32(count_lt);
                } else {
                    const Picked up = pick(umin32(first_above + 1u, len));
                    pb_level = key_to_float(up.key);
                    gap_up = (double)pb_level * (double)positives - (total - up.sum_lt);
                    count_lt = up.count_lt;
                }
                if (count_lt > not_positive) {  // a smaller positive value exists
                    uint32_t down_key = 0u;
                    each([&](float x) __attribute__((always_inline)) {
                        down_key = x > 0.0f && x < pb_level ? umax32(down_key, float_to_key(x)) : down_key;
                    });
                    down_key = wave_max_u32(down_key);
                    float down;
                    double gap_down;
                    if (down_key != 0u) {
                        down = key_to_float(down_key);
                        gap_down = (double)down * (double)positives - (total - smaller_than(down));
                    } else {
                        const Picked below = pick(count_lt);
                        down = key_to_float(below.key);
                        gap_down = (double)down * (double)positives - (total - below.sum_lt);
                    }
                    if (fabs(gap_down) <= fabs(gap_up)) pb_level = down;  // ties take the smaller value
                }
            }
        }
    }

    if constexpr (RULE == kLinear) {
        for (uint32_t k = 1; k + 1 < (uint32_t)S; ++k) {
            const uint32_t rank = 1u + (uint32_t)(((uint64_t)k * (len - 1u)) / (uint32_t)(S - 1));
            const Picked p = pick(rank);
            if (lane == 0u) lds.lvl_value[k] = key_to_float(p.key);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }

    // ---- level solves: greedy recursion (Algorithm 1), then re-solve sweeps ------------------
    [[maybe_unused]] const double bound = RULE == kOptimal ? uniform_f64(lds.sum_error_bound) : 0.0;  // (see floor_t_from_sums)
    if constexpr (S > 2 && S <= 4 && RULE == kOptimal) {
        // Three or four levels: every solve with compile-time level indices and the level records in the
        // wavefront's registers instead of LDS (greedy + S - 2 copies of the routine; with five levels the records no
        // longer fit the 128 registers).
        LevelRecords<S> st;
#pragma unroll
        for (int k = 0; k < S; ++k) {
            st.value[k] = uniform_f32(lds.lvl_value[k]);
            st.rank[k] = 0u;
            st.count_lt[k] = st.count_le[k] = k == S - 1 ? len : 0u;
            st.sum_lt[k] = st.sum_le[k] = k == S - 1 ? uniform_f64(lds.lvl_sum_le[S - 1]) : 0.0;
        }
        auto solve = [&](auto kc, auto lc, auto rc) {
            orq_solve_one_in_registers<decltype(kc)::value, decltype(lc)::value, decltype(rc)::value>(st, lds, pick, len, bound, lane);
        };
        for_greedy_steps<S, 0>(solve);
        for (uint32_t sweep = 0; sweep < sweeps; ++sweep) for_sweep_levels<S, 1>(solve);
        if (lane == 0u) {
#pragma unroll
            for (int k = 1; k < S - 1; ++k) lds.lvl_value[k] = st.value[k];
        }
        wave_lds_sync();
    } else if constexpr (S > 2 && S <= 5 && RULE == kOptimal) {
        // few levels: every solve with compile-time level indices
        auto solve = [&](auto kc, auto lc, auto rc) {
            orq_solve_one(lds, pick, (uint32_t)decltype(kc)::value, (uint32_t)decltype(lc)::value, (uint32_t)decltype(rc)::value,
                          len, bound, lane);
        };
        for_greedy_steps<S, 0>(solve);
        for (uint32_t sweep = 0; sweep < sweeps; ++sweep) for_sweep_levels<S, 1>(solve);
    } else if constexpr (S > 2 && RULE == kOptimal) {
    constexpr GreedyOrder order = greedy_order<S>();
    const uint32_t steps = order.count + sweeps * (S - 2);
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
        orq_solve_one(lds, pick, k, l, r, len, bound, lane);
    }
    }
    return pb_level;
}

template <int C>
struct OrqShape {
    static constexpr int D = 256 * C;               // element capacity of the wave
    static constexpr int B = C >= 16 ? 512 : 256;   // bins
    static constexpr int SHIFT = C >= 16 ? 19 : 20; // magnitude bits dropped: keeps exponent + 4 (3) mantissa bits
};

// FULL: the bucket has exactly 256*C elements (no padding, no per-element validity tests).
// S levels per bucket, BITS bits per level index (S = 2^BITS, or 2^(BITS-1) + 1 for the paper's counts).
template <int C, int S, int BITS, bool FULL, bool CLIP, int RULE>
__device__ __forceinline__ void orq_bucket(OrqLds<OrqShape<C>::D, OrqShape<C>::B, S>& lds, const float* __restrict__ g,
                                           uint32_t len, size_t begin, uint32_t bucket, uint32_t sweeps, float clip,
                                           uint64_t seed, uint64_t index_offset, float* __restrict__ levels,
                                           uint32_t* __restrict__ codes32)
{
    static_assert(S >= 2 && S <= 9 && S <= (1 << BITS), "level count does not fit the index width");
    constexpr int D = OrqShape<C>::D;
    constexpr int B = OrqShape<C>::B;
    constexpr int PER = B / 64;   // bins per lane in the prefix step
    constexpr int HALF = B / 2;   // bins per sign
    constexpr int SHIFT = OrqShape<C>::SHIFT;
    constexpr bool full = FULL;
    constexpr bool PB = RULE == kPb;
    const uint32_t lane = threadIdx.x & 63u;

    // ---- load (past the caches); padding holds NaN and is never binned or encoded ----
    float v[C][4];
    load_range<C, FULL>(v, g, 0u, len, len, lane);

    float limit = __uint_as_float(0x7F800000u);  // clipping threshold
    if (CLIP && clip > 0.0f) {  // (the same for every thread of the grid)
        float(&flat)[4 * C] = reinterpret_cast<float(&)[4 * C]>(v);
        limit = clip_in_registers<4 * C>(flat, len, clip, [&](int j) { return full || (64u * (j & ~3) + 4u * lane + (j & 3) < len); });
        if constexpr (!FULL) set_padding<C>(v, len, lane);
    }

    // ---- extremes ------------------------------------------------------------------------------
    float lane_min, lane_max;
    uint32_t lane_zeros;
    lane_extremes<C, PB>(v, lane_min, lane_max, lane_zeros);
    wave_extremes(lane_min, lane_max);
    const float bucket_min = lane_min + 0.0f, bucket_max = lane_max + 0.0f;  // -0 -> +0
    const uint32_t key_min = float_to_key(bucket_min), key_max = float_to_key(bucket_max);
    const uint32_t mag_max = umax32(__float_as_uint(bucket_min) & 0x7FFFFFFFu, __float_as_uint(bucket_max) & 0x7FFFFFFFu);
    const uint32_t t_max = mag_max >> SHIFT;
    const uint32_t t_low = __builtin_elementwise_sub_sat(t_max, (uint32_t)(HALF - 1));

    float pb_level = 0.0f;
    if constexpr ((S > 2 && RULE != kEven) || PB) {
        // ---- histogram ------------------------------------------------------------------------------
#pragma unroll
        for (int t = 0; t < PER; ++t) lds.bin_start[lane * PER + t] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t slot[C][4];
        count_into_bins<C, FULL, HALF, SHIFT>(slot, v, lds.bin_start, t_low, len, lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        // ---- exclusive prefix over the bin counts (lane l owns bins l*PER .. l*PER+PER-1) ------------
        uint32_t my_start[PER];
        {
            uint32_t cnt[PER];
            uint32_t tot = 0;
#pragma unroll
            for (int t = 0; t < PER; ++t) {
                cnt[t] = lds.bin_start[lane * PER + t];
                tot += cnt[t];
            }
            uint32_t run = wave_inclusive_scan_u32(tot) - tot;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < PER; ++t) {
                my_start[t] = run;
                lds.bin_start[lane * PER + t] = run;
                run += cnt[t];
            }
            if (lane == 63u) lds.bin_start[B] = run;  // = len
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        // ---- scatter the values into their bins ---------------------------------------------------------
        scatter_into_bins<C, FULL>(lds.grouped, &lds.bin_start[HALF], slot, v, 0u, len, lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        // ---- fp64 prefix of the grouped values at block granularity (lane l sums block l) ------------
        // Only the rules whose solves read the counts and sums of picked levels need it: with a single interior
        // level the one solve reads the bucket's total alone, and Linear-s reads nothing.
        constexpr bool SUMS = (RULE == kOptimal && S > 3) || PB;
        {
            double incl = 0.0;
            if constexpr (SUMS) {
                const double part = sum_of_positions<C>(lds.grouped, lane, FULL ? (uint32_t)D : len);
                incl = wave_inclusive_scan_f64(part);
                lds.block_prefix[lane] = incl - part;
            } else if constexpr (RULE == kOptimal) {
                double part = 0.0;
                for_each_chunk<C, FULL>(len, [&](int c, auto all) __attribute__((always_inline)) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const bool valid = decltype(all)::value || (256u * c + 4u * lane + k < len);
                        part += valid ? (double)v[c][k] : 0.0;
                    }
                });
                incl = wave_sum(part);  // the same in every lane
            }
            if (lane == 63u) {
                // the top level is only ever the right end of a solve
                lds.lvl_count_le[S - 1] = len;
                lds.lvl_sum_le[S - 1] = incl;
                lds.lvl_count_lt[S - 1] = len;
                lds.lvl_sum_lt[S - 1] = incl;
            }
        }
        if (lane == 0u) {
            // the bottom level is only ever the left end of a solve
            lds.lvl_count_lt[0] = 0u;
            lds.lvl_sum_lt[0] = 0.0;
            lds.lvl_count_le[0] = 0u;
            lds.lvl_sum_le[0] = 0.0;
        }
        if (lane < (uint32_t)S) {
            lds.lvl_value[lane] = key_to_float(lane == (uint32_t)(S - 1) ? key_max : key_min);
            lds.lvl_rank[lane] = 0u;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        if constexpr (RULE == kOptimal && S > 2) {
            const bool tiny = __ballot(any_tiny_element<HALF, SHIFT>(lds, (uint32_t)D, mag_max, t_low, lane, kWave)) != 0;
            if (lane == 0u) lds.sum_error_bound = tiny ? sum_error_bound_of(mag_max, (uint32_t)D) : 0.0;
            wave_lds_sync();
        }
        const uint32_t zeros = PB ? wave_sum_u32(lane_zeros) : 0u;
        pb_level = orq_solve_levels<S, RULE>(
            lds, [&](uint32_t rank) { return pick_rank<D, B, S, SUMS>(lds, my_start, rank, lane); },
            [&](uint32_t bin) { return __uint_as_float((t_low + (bin - (uint32_t)HALF)) << SHIFT); }, len, zeros, sweeps, lane);
    }

    // every lane holds its own copy of the levels (the selects of the encoder take vector sources)
    float lv[S];
    if constexpr (RULE == kEven) {
        const double largest = (double)__uint_as_float(mag_max);
#pragma unroll
        for (int k = 0; k < S; ++k) lv[k] = (float)(largest * (double)(2 * k - (S - 1)) / (double)(S - 1));
    } else {
        lv[0] = PB ? -pb_level : key_to_float(key_min);
        lv[S - 1] = PB ? pb_level : key_to_float(key_max);
#pragma unroll
        for (int k = 1; k < S - 1; ++k) lv[k] = lds.lvl_value[k];
    }

    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < S; ++k) levels[(size_t)bucket * S + k] = lv[k];
    }

    constexpr bool EVEN = RULE == kEven && S == 3;
    orq_encode<C, S, BITS, FULL, EVEN, EVEN && C == 8 && FULL && !CLIP>(v, lv, len, begin, seed, index_offset, codes32, ReloadFromMemory{g, len, limit},
                                 encoder_table<S, RULE != kEven>(lds.grouped, 0u));
}

// C = 8 (2048-element buckets): 16 buckets fit the LDS of a CU, so the kernel is held to the 128 registers
// that let 4 wavefronts share a SIMD (the clipping variants would otherwise take ~138).
template <int C, int S, int BITS, bool CLIP, int RULE>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(C == 8 ? 4 : 1))) void orq_quantize_kernel(const float* __restrict__ grad, size_t n,
                                                             uint32_t bucket_size, uint32_t sweeps, float clip,
                                                             uint32_t num_buckets, uint64_t seed,
                                                             uint64_t index_offset, float* __restrict__ levels,
                                                             uint32_t* __restrict__ codes32)
{
    __shared__ OrqLds<OrqShape<C>::D, OrqShape<C>::B, S> lds;
    const uint32_t bucket = blockIdx.x;
    if (bucket >= num_buckets) return;
    const size_t begin = (size_t)bucket * bucket_size;
    const size_t rest = n - begin;
    const uint32_t len = rest < bucket_size ? (uint32_t)rest : bucket_size;
    if (len == (uint32_t)OrqShape<C>::D)
        orq_bucket<C, S, BITS, true, CLIP, RULE>(lds, grad + begin, len, begin, bucket, sweeps, clip, seed, index_offset, levels, codes32);
    else
        orq_bucket<C, S, BITS, false, CLIP, RULE>(lds, grad + begin, len, begin, bucket, sweeps, clip, seed, index_offset, levels, codes32);
}

// Clipping when a wavefront holds NB whole buckets (lane l: elements 4l .. 4l+3 of the wavefront's 256, bucket
// l / G with G = 64 / NB): clip_in_registers with the sums taken over the bucket's group of lanes.
template <int NB, bool FULL>
__device__ __forceinline__ void clip_small_buckets(float (&v)[4], uint32_t len, float clip, uint32_t lane)
{
    constexpr uint32_t G = 64u / NB, D = 256u / NB;
    const uint32_t q = lane / G;
    uint32_t count = D;
    if constexpr (!FULL) count = q * D < len ? (len - q * D < D ? len - q * D : D) : 1u;  // (no element: nothing is stored)
    clip_in_registers<4>(
        v, count, clip, [&](int j) { return FULL || 4u * lane + j < len; },
        [&](double& sum, double& squares) __attribute__((always_inline)) {
            auto over_group = [&](double x) __attribute__((always_inline)) {
                x += dpp_f64<kDppXor1>(x);
                x += dpp_f64<kDppXor2>(x);
                x += dpp_f64<kDppHalfMirror>(x);
                x += dpp_f64<kDppMirror>(x);
                if constexpr (G == 32u) {
                    const uint64_t u = (uint64_t)__double_as_longlong(x);
                    const uint32_t lo = lane_xor<16>((uint32_t)u, lane), hi = lane_xor<16>((uint32_t)(u >> 32), lane);
                    x += __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
                }
                return x;
            };
            sum = over_group(sum);
            squares = over_group(squares);
        });
}

// ----------------------------------------------------------------------------------------------
// Evenly spaced levels (QSGD-s, TernGrad) for buckets of 64 or 128 elements: one wavefront takes 256 consecutive
// elements, i.e. NB = 4 or 2 whole buckets (lane l holds elements 4l .. 4l+3, bucket l / G of the wavefront with
// G = 64 / NB lanes per bucket), instead of leaving three quarters or half of its lanes idle.  The only statistic of
// the rule, the largest magnitude, is reduced inside each group of G lanes; every lane then holds the levels of its
// own bucket, which is all the encoder needs.
// ----------------------------------------------------------------------------------------------
template <int S, int BITS, int NB, bool FULL>
__device__ __forceinline__ void even_small_span(const float* __restrict__ g, uint32_t len, size_t begin, uint32_t first_bucket,
                                                float clip, uint64_t seed, uint64_t index_offset,
                                                float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    constexpr uint32_t G = 64u / NB;           // lanes per bucket
    constexpr uint32_t D = 256u / NB;          // elements per bucket
    const uint32_t lane = threadIdx.x & 63u;
    float v[1][4];
    load_range<1, FULL>(v, g, 0u, len, len, lane, 0.0f);
    if (clip > 0.0f) clip_small_buckets<NB, FULL>(v[0], len, clip, lane);
    // largest magnitude of the lane's bucket (padding holds 0)
    uint32_t mag = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) mag = umax32(mag, __float_as_uint(v[0][k]) & 0x7FFFFFFFu);
    mag = umax32(mag, dpp_u32<kDppXor1>(mag));
    mag = umax32(mag, dpp_u32<kDppXor2>(mag));
    mag = umax32(mag, dpp_u32<kDppHalfMirror>(mag));
    mag = umax32(mag, dpp_u32<kDppMirror>(mag));  // the 16 lanes of a row
    if constexpr (G == 32u) mag = umax32(mag, lane_xor<16>(mag, lane));
    float lv[S];
    const double largest = (double)__uint_as_float(mag);
#pragma unroll
    for (int k = 0; k < S; ++k) lv[k] = (float)(largest * (double)(2 * k - (S - 1)) / (double)(S - 1));
    const uint32_t q = lane / G;  // bucket of this lane inside the wavefront
    if (lane % G == 0u && (FULL || q * D < len)) {
#pragma unroll
        for (int k = 0; k < S; ++k) levels[(size_t)(first_bucket + q) * S + k] = lv[k];
    }
    if constexpr (!FULL) set_padding<1>(v, len, lane);
    orq_encode<1, S, BITS, FULL>(v, lv, len, begin, seed, index_offset, codes32, [&](uint32_t, float(&y)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = v[0][k];
    });
}

template <int S, int BITS, int NB>
__global__ __launch_bounds__(4 * kWave) void even_small_kernel(const float* __restrict__ grad, size_t n, float clip,
                                                               uint64_t seed, uint64_t index_offset,
                                                               float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    const size_t span = (size_t)blockIdx.x * 4u + (threadIdx.x >> 6);  // 256 elements each
    const size_t begin = span * 256u;
    if (begin >= n) return;
    const size_t rest = n - begin;
    const uint32_t first_bucket = (uint32_t)(span * NB);
    if (rest >= 256u)
        even_small_span<S, BITS, NB, true>(grad + begin, 256u, begin, first_bucket, clip, seed, index_offset, levels, codes32);
    else
        even_small_span<S, BITS, NB, false>(grad + begin, (uint32_t)rest, begin, first_bucket, clip, seed, index_offset, levels,
                                            codes32);
}

// ----------------------------------------------------------------------------------------------
// ORQ, Linear-s and BinGrad-pb for buckets of 64 or 128 elements, NB = 4 or 2 whole buckets per wavefront in the
// layout of even_small_span.  A bucket this small is not grouped into bins: its 4 G keys (G = 64 / NB lanes, 4 registers
// each) are sorted in registers by a bitonic network whose every compare-exchange is ascending -- the first step of
// a merge pairs element e with e ^ (run length - 1), i.e. reverses the second run -- so that no step needs a
// direction.  Element e = 4 * (lane inside the bucket) + register.  The levels are then order statistics fetched
// from the sorted registers: the extremes, and either Linear-s's ranks or the elements of the ranks that the optimal
// condition asks for.  With three levels there is one solve, between the extremes, and it reads the bucket's total
// alone (sweeps repeat it unchanged); with more, every lane keeps the level records of its bucket and the solves of
// all buckets of the wavefront run side by side.  Two levels are the extremes and need no sort.  BinGrad-pb's level
// is the positive value at the sign change of its condition, which every element evaluates for itself from the
// exclusive fp64 prefix of the sorted values.
// ----------------------------------------------------------------------------------------------
__device__ __forceinline__ void sort_pair(uint32_t& a, uint32_t& b)
{
    const uint32_t mn = umin32(a, b), mx = umax32(a, b);
    a = mn;
    b = mx;
}

// The steps of a merge that pair lanes J apart (J = M / 2 ... 1), register by register.
template <int J>
__device__ __forceinline__ void row_sort_across(uint32_t (&x)[4], uint32_t lane)
{
    if constexpr (J >= 1) {
        const uint32_t bound = upper_lanes<J>(lane);
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = smaller_or_larger(x[r], lane_xor<J>(x[r], lane), bound);
        row_sort_across<J / 2>(x, lane);
    }
}

// Merges the sorted runs of 4 M elements (M lanes) pairwise into sorted runs of 8 M, and so on up to 4 G.
template <int M, int G>
__device__ __forceinline__ void row_sort_merge(uint32_t (&x)[4], uint32_t lane)
{
    if constexpr (2 * M <= G) {
        const uint32_t bound = upper_lanes<M>(lane);
        uint32_t y[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) y[r] = lane_reverse<M>(x[3 - r], lane);
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = smaller_or_larger(x[r], y[r], bound);
        row_sort_across<M / 2>(x, lane);
        sort_pair(x[0], x[2]);
        sort_pair(x[1], x[3]);
        sort_pair(x[0], x[1]);
        sort_pair(x[2], x[3]);
        row_sort_merge<2 * M, G>(x, lane);
    }
}

// Ascending sort of the 4 G keys of every group of G lanes (G = 16 or 32).
template <int G>
__device__ __forceinline__ void row_sort(uint32_t (&x)[4], uint32_t lane)
{
    sort_pair(x[0], x[1]);  // runs of 2
    sort_pair(x[2], x[3]);
    sort_pair(x[0], x[3]);  // runs of 4
    sort_pair(x[1], x[2]);
    sort_pair(x[0], x[1]);
    sort_pair(x[2], x[3]);
    row_sort_merge<1, G>(x, lane);
}

// Element `index` (0-based, the same in all lanes of the group) of the sorted group whose first lane is `first_lane`.
__device__ __forceinline__ uint32_t row_fetch(const uint32_t (&x)[4], uint32_t index, uint32_t first_lane)
{
    const uint32_t lo = (index & 1u) ? x[1] : x[0];
    const uint32_t hi = (index & 1u) ? x[3] : x[2];
    const uint32_t mine = (index & 2u) ? hi : lo;
    return (uint32_t)__builtin_amdgcn_ds_bpermute((int)((first_lane + (index >> 2)) << 2), (int)mine);
}

// Sum over the group of G = 8, 16 or 32 lanes, in every lane of the group.
template <int G>
__device__ __forceinline__ double row_sum_f64(double x, uint32_t lane)
{
    x += dpp_f64<kDppXor1>(x);
    x += dpp_f64<kDppXor2>(x);
    x += dpp_f64<kDppHalfMirror>(x);
    if constexpr (G >= 16) x += dpp_f64<kDppMirror>(x);
    if constexpr (G == 32) {
        const uint64_t u = (uint64_t)__double_as_longlong(x);
        const uint32_t lo = lane_xor<16>((uint32_t)u, lane), hi = lane_xor<16>((uint32_t)(u >> 32), lane);
        x += __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    }
    return x;
}

template <int G>
__device__ __forceinline__ uint32_t row_sum_u32(uint32_t x, uint32_t lane)
{
    x += dpp_u32<kDppXor1>(x);
    x += dpp_u32<kDppXor2>(x);
    x += dpp_u32<kDppHalfMirror>(x);
    if constexpr (G >= 16) x += dpp_u32<kDppMirror>(x);
    if constexpr (G == 32) x += lane_xor<16>(x, lane);
    return x;
}

// Minimum over the group of G lanes, in every lane of the group.
template <int G>
__device__ __forceinline__ uint32_t row_min_u32(uint32_t x, uint32_t lane)
{
    x = umin32(x, dpp_u32<kDppXor1>(x));
    x = umin32(x, dpp_u32<kDppXor2>(x));
    x = umin32(x, dpp_u32<kDppHalfMirror>(x));
    if constexpr (G >= 16) x = umin32(x, dpp_u32<kDppMirror>(x));
    if constexpr (G == 32) x = umin32(x, lane_xor<16>(x, lane));
    return x;
}

template <int G>
__device__ __forceinline__ uint32_t row_max_u32(uint32_t x, uint32_t lane)
{
    return ~row_min_u32<G>(~x, lane);
}

// Inclusive scan over the lanes of every group of G lanes (G = 16 or 32).
template <int G>
__device__ __forceinline__ double row_inclusive_scan_f64(double x)
{
    x += dpp_or_zero_f64<kDppRowShr1, 0xF>(x);
    x += dpp_or_zero_f64<kDppRowShr2, 0xF>(x);
    x += dpp_or_zero_f64<kDppRowShr4, 0xF>(x);
    x += dpp_or_zero_f64<kDppRowShr8, 0xF>(x);
    if constexpr (G == 32) x += dpp_or_zero_f64<kDppRowBcast15, 0xA>(x);
    return x;
}

__device__ __forceinline__ double lane_fetch_f64(double x, uint32_t from_lane)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(from_lane << 2), (int)(uint32_t)u);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(from_lane << 2), (int)(uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// row_fetch for the fp64 sums that sit beside the sorted keys.
__device__ __forceinline__ double row_fetch_f64(const double (&x)[4], uint32_t index, uint32_t first_lane)
{
    const double lo = (index & 1u) ? x[1] : x[0];
    const double hi = (index & 1u) ? x[3] : x[2];
    return lane_fetch_f64((index & 2u) ? hi : lo, first_lane + (index >> 2));
}

// Per level, in the registers of every lane of the bucket's group: what OrqLds keeps per level.
template <int S>
struct RowLevels {
    float value[S];
    uint32_t count_lt[S], count_le[S], rank[S];
    double sum_lt[S], sum_le[S];
};

template <int S, int BITS, int NB, bool FULL, int RULE>
__device__ __forceinline__ void sorted_small_span(const float* __restrict__ g, uint32_t len, size_t begin, uint32_t first_bucket,
                                                  uint32_t sweeps, float clip, uint64_t seed, uint64_t index_offset,
                                                  float* __restrict__ levels, uint32_t* __restrict__ codes32,
                                                  unsigned long long* exact_limbs)
{
    static_assert(RULE == kLinear || RULE == kOptimal || (RULE == kPb && S == 2), "rules that read order statistics");
    constexpr uint32_t G = 64u / NB;  // lanes per bucket
    constexpr uint32_t D = 256u / NB;  // elements per bucket
    const uint32_t lane = threadIdx.x & 63u;
    float v[1][4];
    load_range<1, FULL>(v, g, 0u, len, len, lane, 0.0f);
    if (clip > 0.0f) clip_small_buckets<NB, FULL>(v[0], len, clip, lane);
    const uint32_t q = lane / G;  // bucket of this lane inside the wavefront
    uint32_t count = D;           // elements of that bucket (the gradient may end inside or before it)
    if constexpr (!FULL) count = q * D < len ? (len - q * D < D ? len - q * D : D) : 0u;

    uint32_t x[4];
    double part = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const bool valid = FULL || 4u * lane + k < len;
        const float value = v[0][k] + 0.0f;  // -0 -> +0
        x[k] = valid ? float_to_key(value) : 0xFFFFFFFFu;  // padding sorts behind every value
        if constexpr (RULE == kOptimal && S == 3) part += valid ? (double)value : 0.0;
    }
    float lv[S];
    if constexpr (RULE == kPb) {
        // b_1 minimises |b * #{v > 0} - sum_{v >= b} v| over the bucket's positive values.  Every element evaluates the
        // difference for its own value in its own lane (the sum of the smaller elements is its entry of the exclusive
        // prefix if it is the first of its value); the difference grows with b, so the minimiser is the first value
        // where it is not negative, or the distinct value just below.
        row_sort<(int)G>(x, lane);
        const uint32_t first_lane = lane & ~(G - 1u);
        const uint32_t l4 = 4u * (lane & (G - 1u));
        constexpr uint32_t kZeroKey = 0x80000000u;  // key of +0
        double before[4], run = 0.0;
        uint32_t not_positive = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            before[r] = run;
            run += l4 + r < count ? (double)key_to_float(x[r]) : 0.0;
            not_positive += x[r] <= kZeroKey ? 1u : 0u;
        }
        const double incl = row_inclusive_scan_f64<(int)G>(run);
        const double lanes_before = incl - run;
        const double total = lane_fetch_f64(incl, first_lane + G - 1u);
        not_positive = row_sum_u32<(int)G>(not_positive, lane);
        const uint32_t positives = count - (not_positive < count ? not_positive : count);
        // last key of the lane in front (none for the first lane of the group: key 0 lies below every positive key)
        const uint32_t front = (uint32_t)__builtin_amdgcn_ds_bpermute((int)((lane - 1u) << 2), (int)x[3]);
        double gap[4];
        uint32_t first_ok = 0xFFFFu, last_first = 0u;  // element indices inside the bucket
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            before[r] += lanes_before;
            const uint32_t previous = r > 0 ? x[r > 0 ? r - 1 : 0] : (lane == first_lane ? 0u : front);
            const bool candidate = l4 + r < count && x[r] > kZeroKey && x[r] != previous;  // first of a positive value
            gap[r] = (double)key_to_float(x[r]) * (double)positives - (total - before[r]);
            if (candidate && gap[r] >= 0.0) first_ok = umin32(first_ok, l4 + r);
            if (candidate) last_first = umax32(last_first, l4 + r);
        }
        first_ok = row_min_u32<(int)G>(first_ok, lane);
        last_first = row_max_u32<(int)G>(last_first, lane);
        // (the largest value's difference is >= 0 but for rounding: if no element says so, it is the answer)
        const uint32_t at = first_ok != 0xFFFFu ? first_ok : last_first;
        const float up = key_to_float(row_fetch(x, at, first_lane));
        const double gap_up = row_fetch_f64(gap, at, first_lane);
        // the distinct value just below, which counts if it is positive: its difference sits where that value begins
        const uint32_t down_key = row_fetch(x, at > 0u ? at - 1u : 0u, first_lane);
        uint32_t down_at = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) down_at += x[r] < down_key ? 1u : 0u;
        down_at = row_sum_u32<(int)G>(down_at, lane);
        const double gap_down = row_fetch_f64(gap, down_at, first_lane);
        const bool take_down = at > not_positive && fabs(gap_down) <= fabs(gap_up);  // ties take the smaller value
        const float pb_level = positives > 0u ? (take_down ? key_to_float(down_key) : up) : 0.0f;
        lv[0] = -pb_level;
        lv[1] = pb_level;
    } else if constexpr (S == 2) {
        // two levels are the extremes: no sort, two reductions over the group
        uint32_t low = umin32(umin32(x[0], x[1]), umin32(x[2], x[3])), high = 0u;
#pragma unroll
        for (int k = 0; k < 4; ++k) high = umax32(high, x[k] == 0xFFFFFFFFu ? 0u : x[k]);
        lv[0] = key_to_float(row_min_u32<(int)G>(low, lane));
        lv[1] = key_to_float(row_max_u32<(int)G>(high, lane));
    } else {
        row_sort<(int)G>(x, lane);

        const uint32_t first_lane = lane & ~(G - 1u);
        const uint32_t last = count > 0u ? count - 1u : 0u;
        lv[0] = key_to_float(row_fetch(x, 0u, first_lane));
        lv[S - 1] = key_to_float(row_fetch(x, last, first_lane));
        // Whether the fp64 sums of this lane's bucket are exact (floor_t_from_sums: no non-zero element more than
        // safe_binades(D) binades below the largest magnitude), and the bucket's workspace for exact_floor_t.
        double error_bound = 0.0;
        unsigned long long* limb = exact_limbs + ((threadIdx.x >> 6) * NB + q) * kExactLimbs;
        if constexpr (RULE == kOptimal) {
            const uint32_t mag_max = umax32(__float_as_uint(lv[0]) & 0x7FFFFFFFu, __float_as_uint(lv[S - 1]) & 0x7FFFFFFFu);
            const uint32_t biased = mag_max >> 23;
            const uint32_t mag_safe = biased > safe_binades(D) ? (biased - safe_binades(D)) << 23 : 0u;
            uint32_t tiny = 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t magnitude = __float_as_uint(key_to_float(x[i])) & 0x7FFFFFFFu;
                if (4u * (lane & (G - 1u)) + i < count && magnitude != 0u && magnitude < mag_safe) tiny = 1u;
            }
            if (row_max_u32<(int)G>(tiny, lane) != 0u) error_bound = sum_error_bound_of(mag_max, D);
        }
        if constexpr (RULE == kLinear) {
#pragma unroll
            for (int k = 1; k + 1 < S; ++k)
                lv[k] = key_to_float(row_fetch(x, ((uint32_t)k * last) / (uint32_t)(S - 1), first_lane));
        } else if constexpr (S > 3) {
            // The solves of orq_solve_levels, every lane keeping the records of its own bucket.  What a solve needs
            // around a picked element comes from the sorted registers: the counts of smaller and of not larger keys
            // (summed over the group), and the sum of the smaller ones, an entry of the exclusive fp64 prefix.
            const uint32_t l4 = 4u * (lane & (G - 1u));
            double before[4];  // sum of the sorted elements in front of element 4 l + r
            double total;
            {
                double run = 0.0, mine[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    mine[r] = run;
                    run += l4 + r < count ? (double)key_to_float(x[r]) : 0.0;
                }
                const double incl = row_inclusive_scan_f64<(int)G>(run);
                const double lanes_before = incl - run;
#pragma unroll
                for (int r = 0; r < 4; ++r) before[r] = lanes_before + mine[r];
                total = lane_fetch_f64(incl, first_lane + G - 1u);
            }
            RowLevels<S> st;
#pragma unroll
            for (int k = 0; k < S; ++k) {
                st.value[k] = k == S - 1 ? lv[S - 1] : lv[0];
                st.count_lt[k] = k == S - 1 ? count : 0u;
                st.count_le[k] = k == S - 1 ? count : 0u;
                st.sum_lt[k] = k == S - 1 ? total : 0.0;
                st.sum_le[k] = k == S - 1 ? total : 0.0;
                st.rank[k] = 0u;
            }
            const uint32_t count_or_one = count > 0u ? count : 1u;
            auto solve = [&](auto kc, auto lc, auto rc) {
                constexpr int k = decltype(kc)::value, l = decltype(lc)::value, r = decltype(rc)::value;
                const float L = st.value[l], R = st.value[r];
                const uint32_t cnt_lt_L = st.count_lt[l], cnt_le_R = st.count_le[r];
                const double sum_lt_L = st.sum_lt[l], sum_le_R = st.sum_le[r];
                const bool ordered = L < R;
                // S = sum_{L<=v<=R} (v - L),  T = S / (R - L),  level = element of rank #{v<=R} - floor(T)
                const uint32_t count_in = cnt_le_R - cnt_lt_L;
                const double Ssum = (sum_le_R - sum_lt_L) - (double)L * (double)count_in;
                const double width = (double)R - (double)L;
                double m;  // not used when L == R
                const bool decided = floor_t_from_sums(Ssum, width, error_bound, m);
                if (ordered && !decided) {
                    // (as in orq_solve_one: exact sums where the fp64 sums do not decide; only the lanes of such buckets)
                    m = (double)exact_floor_t_registers(limb, lane & (G - 1u), L, R, count_in, (uint32_t)m, key_to_float(x[0]),
                                                        key_to_float(x[1]), key_to_float(x[2]), key_to_float(x[3]),
                                                        count > l4 ? count - l4 : 0u);
                }
                const bool whole = m >= (double)cnt_le_R;
                uint32_t rank = whole ? 1u : cnt_le_R - (uint32_t)(whole ? 0.0 : m);
                rank = rank < 1u ? 1u : (rank > count_or_one ? count_or_one : rank);
                const bool same = ordered && rank == st.rank[k];  // same element as last time
                if (__ballot(!same) == 0) return;
                const uint32_t key = row_fetch(x, rank - 1u, first_lane);
                const float picked = key_to_float(key);
                uint32_t below = 0, not_above = 0;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    below += x[i] < key ? 1u : 0u;
                    not_above += x[i] <= key ? 1u : 0u;
                }
                const uint32_t both = row_sum_u32<(int)G>(below | (not_above << 16), lane);  // two counts of at most 128
                const uint32_t c_lt = both & 0xFFFFu, c_le = both >> 16;
                const double s_lt = row_fetch_f64(before, c_lt, first_lane);
                const double s_le = s_lt + (double)(c_le - c_lt) * (double)picked;
                const bool copy_left = !ordered || picked < L;  // the level coincides with the left end
                const float new_value = copy_left ? L : picked;
                const uint32_t new_count_lt = copy_left ? cnt_lt_L : c_lt;
                const double new_sum_lt = copy_left ? sum_lt_L : s_lt;
                const uint32_t new_count_le = copy_left ? (ordered ? st.count_le[l] : cnt_le_R) : c_le;
                const double new_sum_le = copy_left ? (ordered ? st.sum_le[l] : sum_le_R) : s_le;
                const uint32_t new_rank = copy_left ? 0u : rank;
                st.value[k] = same ? st.value[k] : new_value;
                st.count_lt[k] = same ? st.count_lt[k] : new_count_lt;
                st.sum_lt[k] = same ? st.sum_lt[k] : new_sum_lt;
                st.count_le[k] = same ? st.count_le[k] : new_count_le;
                st.sum_le[k] = same ? st.sum_le[k] : new_sum_le;
                st.rank[k] = same ? st.rank[k] : new_rank;
            };
            for_greedy_steps<S, 0>(solve);
            for (uint32_t sweep = 0; sweep < sweeps; ++sweep) for_sweep_levels<S, 1>(solve);
#pragma unroll
            for (int k = 1; k + 1 < S; ++k) lv[k] = st.value[k];
        } else {
            // S = sum (v - L) over the bucket, T = S / (R - L), level = element of rank #{v <= R} - floor(T)
            const double total = row_sum_f64<(int)G>(part, lane);
            const float L = lv[0], R = lv[2];
            const double Ssum = total - (double)L * (double)count, width = (double)R - (double)L;
            double m;  // not used when L == R
            const bool decided = floor_t_from_sums(Ssum, width, error_bound, m);
            if (L < R && !decided) {
                // (as in orq_solve_one: exact sums where the fp64 sums do not decide; only the lanes of such buckets)
                const uint32_t mine = 4u * (lane & (G - 1u));
                m = (double)exact_floor_t_registers(limb, lane & (G - 1u), L, R, count, (uint32_t)m, key_to_float(x[0]),
                                                    key_to_float(x[1]), key_to_float(x[2]), key_to_float(x[3]),
                                                    count > mine ? count - mine : 0u);
            }
            if (m > (double)count) m = (double)count;
            uint32_t rank = m >= (double)count ? 1u : count - (uint32_t)m;
            rank = rank < 1u ? 1u : rank;
            const float picked = key_to_float(row_fetch(x, rank - 1u, first_lane));
            lv[1] = (L < R && !(picked < L)) ? picked : L;
        }
    }
    if (lane % G == 0u && (FULL || q * D < len)) {
#pragma unroll
        for (int k = 0; k < S; ++k) levels[(size_t)(first_bucket + q) * S + k] = lv[k];
    }
    if constexpr (!FULL) set_padding<1>(v, len, lane);
    orq_encode<1, S, BITS, FULL>(v, lv, len, begin, seed, index_offset, codes32, [&](uint32_t, float(&y)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) y[k] = v[0][k];
    });
}

template <int S, int BITS, int NB, int RULE>
__global__ __launch_bounds__(4 * kWave) void sorted_small_kernel(const float* __restrict__ grad, size_t n, uint32_t sweeps,
                                                                 float clip, uint64_t seed, uint64_t index_offset,
                                                                 float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    __shared__ unsigned long long exact_limbs[4 * NB * kExactLimbs];  // workspace of exact_floor_t per wavefront and bucket
    const size_t span = (size_t)blockIdx.x * 4u + (threadIdx.x >> 6);  // 256 elements each
    const size_t begin = span * 256u;
    if (begin >= n) return;
    const size_t rest = n - begin;
    const uint32_t first_bucket = (uint32_t)(span * NB);
    if (rest >= 256u)
        sorted_small_span<S, BITS, NB, true, RULE>(grad + begin, 256u, begin, first_bucket, sweeps, clip, seed, index_offset,
                                                   levels, codes32, exact_limbs);
    else
        sorted_small_span<S, BITS, NB, false, RULE>(grad + begin, (uint32_t)rest, begin, first_bucket, sweeps, clip, seed,
                                                    index_offset, levels, codes32, exact_limbs);
}

// ----------------------------------------------------------------------------------------------
// ORQ and the other random-rounding rules with W = 2 .. 16 wavefronts of a workgroup owning one bucket (up
// to 32768 elements), wavefront w holding bucket elements [256 C w, 256 C (w + 1)) in the register layout of
// orq_bucket.  All of them build the grouping of the whole bucket in LDS (histogram, bin
// starts, scatter, fp64 block prefix) with workgroup barriers in between; the level solves run on wavefront 0, those of
// five and more levels on the first two (orq_team_solve); then every wavefront encodes its own elements.
//
// What bounds it: with few buckets the latency of one; with many (buckets above 4096 elements) the solves, a step of which ends in
// a barrier and spends 64 lanes on one scalar chain (buckets up to 4096 elements: pool_kernels.h).
// ----------------------------------------------------------------------------------------------
template <int W, int C>
struct alignas(16) OrqTeamLds {
    static constexpr int D = 256 * C * W;
    // bins, and magnitude bits dropped by the bin index (what is kept: the exponent and 3 .. 6 mantissa bits)
    static constexpr int B = D >= 16384 ? 2048 : D >= 8192 ? 1024 : D >= 4096 ? 512 : 256;
    static constexpr int SHIFT = D >= 16384 ? 17 : D >= 8192 ? 18 : D >= 4096 ? 19 : 20;
    static constexpr int BLOCK = C < 8 ? 32 : 4 * C;  // positions per entry of the fp64 block prefix
    uint32_t grouped[D];
    uint32_t bin_start[B + 4];
    double block_prefix[D / BLOCK];  // fp64 sum of all positions before block i of BLOCK positions
    double lvl_sum_lt[10];
    double lvl_sum_le[10];
    float lvl_value[10];
    uint32_t lvl_count_lt[10];
    uint32_t lvl_count_le[10];
    uint32_t lvl_rank[10];
    double sum_error_bound;  // 0 when every fp64 sum of the bucket is exact (see floor_t_from_sums)
    uint32_t tiny_flag;      // set by any thread that met an element too small for exact sums
    unsigned long long exact_limb[2][kExactLimbs];  // workspace of exact_floor_t, one per solving wavefront
    TeamSlot slots[2][W];
};

template <int W, int C, int S, int BITS, bool FULL, int RULE>
__device__ __forceinline__ void orq_team_bucket(OrqTeamLds<W, C>& lds, const float* __restrict__ g, uint32_t len,
                                                size_t begin, uint32_t bucket, uint32_t sweeps, float clip,
                                                uint64_t seed, uint64_t index_offset, float* __restrict__ levels,
                                                uint32_t* __restrict__ codes32)
{
    constexpr uint32_t PER_WAVE = 256u * C;  // bucket elements per wavefront
    constexpr int B = OrqTeamLds<W, C>::B;
    constexpr int HALF = B / 2;
    constexpr int SHIFT = OrqTeamLds<W, C>::SHIFT;
    constexpr bool PB = RULE == kPb;
    constexpr uint32_t THREADS = 64u * W;
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = uniform_u32(tid >> 6);
    const uint32_t first = PER_WAVE * wave;  // first bucket element of this wavefront
    const uint32_t my_len = len > first ? (len - first < PER_WAVE ? len - first : PER_WAVE) : 0u;
    WaveTeam<W> team{lds.slots, wave, 0u};

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

    // ---- extremes of the whole bucket ----------------------------------------------------------------
    float lane_min, lane_max;
    uint32_t lane_zeros;
    lane_extremes<C, PB>(v, lane_min, lane_max, lane_zeros);
    wave_extremes(lane_min, lane_max);
    float bucket_min = lane_min, bucket_max = lane_max;
    uint32_t zeros = PB ? wave_sum_u32(lane_zeros) : 0u;
    {
        const TeamSlot* s = team.exchange((double)zeros, __float_as_uint(bucket_min), __float_as_uint(bucket_max));
        double z = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            bucket_min = fminf(bucket_min, __uint_as_float(s[w].a));
            bucket_max = fmaxf(bucket_max, __uint_as_float(s[w].b));
            z += s[w].sum;
        }
        zeros = (uint32_t)z;
    }
    bucket_min += 0.0f;  // -0 -> +0
    bucket_max += 0.0f;
    const uint32_t key_min = float_to_key(bucket_min), key_max = float_to_key(bucket_max);
    const uint32_t mag_max = umax32(__float_as_uint(bucket_min) & 0x7FFFFFFFu, __float_as_uint(bucket_max) & 0x7FFFFFFFu);
    const uint32_t t_max = mag_max >> SHIFT;
    const uint32_t t_low = __builtin_elementwise_sub_sat(t_max, (uint32_t)(HALF - 1));

    if constexpr ((S > 2 && RULE != kEven) || PB) {
        // ---- histogram --------------------------------------------------------------------------------
        for (uint32_t i = tid; i < (uint32_t)B; i += THREADS) lds.bin_start[i] = 0u;
        if (tid == 0u) lds.tiny_flag = 0u;
        __syncthreads();
        uint32_t slot[C][4];
        count_into_bins<C, FULL, HALF, SHIFT>(slot, v, lds.bin_start, t_low, my_len, lane);
        __syncthreads();

        // ---- exclusive prefix over the bin counts --------------------------------------------------------
        // Wavefront 0, lane l owning bins l*PER .. l*PER+PER-1; 2048 bins: all wavefronts, thread t owning bins t*PER .. likewise.  32 bins to a lane
        // are 32 registers on top of the values and their slots, which eight wavefronts of 2048 elements do not have: 76 to 80 bytes per lane went to
        // scratch memory, and Linear-5 in 1628 buckets of 12288 took 60.1 us where it takes 51.8 now (four levels, two sweeps, 1000 of 24576 102.3 -> 98.9).
        // Linear-s with 4096 elements per wavefront, which has the registers, is 1.5 to 2 % faster with one (700 buckets of 28672 66.9 and 68.0).
        if constexpr (B >= 2048 && (C == 8 || RULE != kLinear)) {
            constexpr uint32_t PER = B / THREADS;
            uint32_t count[PER], tot = 0;
#pragma unroll
            for (uint32_t i = 0; i < PER; ++i) {
                count[i] = lds.bin_start[tid * PER + i];
                tot += count[i];
            }
            const uint32_t incl = wave_inclusive_scan_u32(tot);
            const TeamSlot* s = team.exchange(0.0, __builtin_amdgcn_readlane(incl, 63), 0u);
            uint32_t run = incl - tot;
#pragma unroll
            for (int w = 0; w < W; ++w) run += (uint32_t)w < wave ? s[w].a : 0u;
#pragma unroll
            for (uint32_t i = 0; i < PER; ++i) {
                lds.bin_start[tid * PER + i] = run;
                run += count[i];
            }
            if (tid == THREADS - 1u) lds.bin_start[B] = run;  // = len
        } else if (wave == 0u) {
            constexpr uint32_t PER = B / 64;
            uint32_t tot = 0;
            for (uint32_t i = 0; i < PER; ++i) tot += lds.bin_start[lane * PER + i];
            uint32_t run = wave_inclusive_scan_u32(tot) - tot;
            for (uint32_t i = 0; i < PER; ++i) {
                const uint32_t count = lds.bin_start[lane * PER + i];
                lds.bin_start[lane * PER + i] = run;
                run += count;
            }
            if (lane == 63u) lds.bin_start[B] = run;  // = len
        }
        __syncthreads();

        // ---- scatter the values into their bins ---------------------------------------------------------
        scatter_into_bins<C, FULL>(lds.grouped, &lds.bin_start[HALF], slot, v, first, my_len, lane);
        __syncthreads();

        // ---- may the fp64 sums round?  (all threads look; combined before the records below are written) ----
        if constexpr (RULE == kOptimal && S > 2) {
            if (any_tiny_element<HALF, SHIFT>(lds, (uint32_t)OrqTeamLds<W, C>::D, mag_max, t_low, tid, THREADS))
                atomicOr(&lds.tiny_flag, 1u);
        }

        // ---- fp64 prefix of the grouped values (thread t sums positions [4C t, 4C (t + 1))) ------------------
        // Skipped, but for the bucket's total, by the rules whose solves read no picked level's counts or sums.
        constexpr bool SUMS = (RULE == kOptimal && S > 3) || PB;
        {
            double total = 0.0;
            if constexpr (SUMS) {
                constexpr uint32_t SPANS = OrqTeamLds<W, C>::BLOCK / (4u * C);
                const double part = sum_of_positions<C>(lds.grouped, tid, FULL ? (uint32_t)OrqTeamLds<W, C>::D : len);
                const double incl = wave_inclusive_scan_f64(part);
                const TeamSlot* s = team.exchange(readlane_f64(incl, 63), 0u, 0u);
                double before = 0.0;
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    if ((uint32_t)w < wave) before += s[w].sum;
                    total += s[w].sum;
                }
                if (tid % SPANS == 0u) lds.block_prefix[tid / SPANS] = before + (incl - part);
            } else if constexpr (RULE == kOptimal) {
                double part = 0.0;
                for_each_chunk<C, FULL>(my_len, [&](int c, auto all) __attribute__((always_inline)) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const bool valid = decltype(all)::value || (256u * c + 4u * lane + k < my_len);
                        part += valid ? (double)v[c][k] : 0.0;
                    }
                });
                const TeamSlot* s = team.exchange(wave_sum(part), 0u, 0u);
#pragma unroll
                for (int w = 0; w < W; ++w) total += s[w].sum;
            }
            if (tid == 0u) {
                // the bottom level is only ever the left end of a solve, the top level the right end
                lds.lvl_count_lt[0] = 0u;
                lds.lvl_sum_lt[0] = 0.0;
                lds.lvl_count_le[0] = 0u;
                lds.lvl_sum_le[0] = 0.0;
                lds.lvl_count_le[S - 1] = len;
                lds.lvl_sum_le[S - 1] = total;
                lds.lvl_count_lt[S - 1] = len;
                lds.lvl_sum_lt[S - 1] = total;
                // (every thread's look at the small elements lies before the barrier of the exchange above)
                if constexpr (RULE == kOptimal && S > 2)
                    lds.sum_error_bound = lds.tiny_flag != 0u ? sum_error_bound_of(mag_max, (uint32_t)OrqTeamLds<W, C>::D) : 0.0;
            }
            if (tid < (uint32_t)S) {
                lds.lvl_value[tid] = key_to_float(tid == (uint32_t)(S - 1) ? key_max : key_min);
                lds.lvl_rank[tid] = 0u;
            }
        }
        __syncthreads();

        if constexpr (RULE == kOptimal && S > 2) {
            // ---- the level solves, spread over the first two wavefronts ------------------------------------------
            // Up to four levels there is next to nothing to spread: wavefront 0 alone, with the records in its registers
            // and no barrier per step (ORQ-4, 25.6 M values in buckets of 4096: 61 -> 55 us).
            auto pick = [&](uint32_t rank) { return pick_rank_by_lookup<SUMS>(lds, rank, lane); };
            if constexpr (S <= 4) {
                if (wave == 0u) orq_solve_levels<S, RULE>(lds, pick, [](uint32_t) { return 0.0f; }, len, 0u, sweeps, lane);
                __syncthreads();
            } else {
                orq_team_solve<S>(lds, pick, wave, len, sweeps, lane);
            }
        } else {
            // ---- the other rules' solves are serial: wavefront 0 ---------------------------------------------------
            if (wave == 0u) {
                const float pb_level = orq_solve_levels<S, RULE>(
                    lds, [&](uint32_t rank) { return pick_rank_by_lookup<SUMS>(lds, rank, lane); },
                    [&](uint32_t bin) { return __uint_as_float((t_low + (bin - (uint32_t)HALF)) << SHIFT); }, len, zeros, sweeps,
                    lane);
                if (PB && lane == 0u) {
                    lds.lvl_value[0] = -pb_level;
                    lds.lvl_value[S - 1] = pb_level;
                }
            }
            __syncthreads();
        }
    }

    float lv[S];
    if constexpr (RULE == kEven) {
        const double largest = (double)__uint_as_float(mag_max);
#pragma unroll
        for (int k = 0; k < S; ++k) lv[k] = (float)(largest * (double)(2 * k - (S - 1)) / (double)(S - 1));
    } else if constexpr (S == 2 && !PB) {
        lv[0] = key_to_float(key_min);
        lv[1] = key_to_float(key_max);
    } else {
#pragma unroll
        for (int k = 0; k < S; ++k) lv[k] = lds.lvl_value[k];
    }
    if (tid == 0u) {
#pragma unroll
        for (int k = 0; k < S; ++k) levels[(size_t)bucket * S + k] = lv[k];
    }

    orq_encode<C, S, BITS, FULL, RULE == kEven && S == 3>(v, lv, my_len, begin + first, seed, index_offset, codes32, ReloadFromMemory{g + first, my_len, limit},
                                 encoder_table<S, RULE != kEven>(lds.grouped, wave));
}

// C = 8 (2048 elements per wavefront): the LDS of a CU holds the buckets of 16 wavefronts, so the kernel is held to the
// 128 registers that let four wavefronts share a SIMD (one register more costs d = 8192 a quarter of its wavefronts);
// BinGrad-pb would spill.  W = C = 4: to the 72 registers that seven wavefronts can have.
template <int W, int C, int S, int BITS, int RULE>
__global__ __launch_bounds__(W* kWave) __attribute__((amdgpu_waves_per_eu(RULE == kPb ? 1 : C == 8 ? 4 : C == 4 && W == 4 ? 7 : 1))) void orq_team_kernel(const float* __restrict__ grad, size_t n,
                                                            uint32_t bucket_size, uint32_t sweeps, float clip,
                                                            uint32_t num_buckets, uint64_t seed, uint64_t index_offset,
                                                            float* __restrict__ levels, uint32_t* __restrict__ codes32)
{
    __shared__ OrqTeamLds<W, C> lds;
    const uint32_t bucket = blockIdx.x;
    if (bucket >= num_buckets) return;
    const size_t begin = (size_t)bucket * bucket_size;
    const size_t rest = n - begin;
    const uint32_t len = rest < bucket_size ? (uint32_t)rest : bucket_size;
    if (len == (uint32_t)OrqTeamLds<W, C>::D)
        orq_team_bucket<W, C, S, BITS, true, RULE>(lds, grad + begin, len, begin, bucket, sweeps, clip, seed, index_offset, levels, codes32);
    else
        orq_team_bucket<W, C, S, BITS, false, RULE>(lds, grad + begin, len, begin, bucket, sweeps, clip, seed, index_offset, levels, codes32);
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------
// Which rules and level counts the dispatch in rounding_part.hip gives to one wavefront of 256 C elements per bucket, and (below) to
// W wavefronts.  The others are not compiled, and asking for one fails like a launch that the runtime refuses: a call must not
// return success over outputs that nothing has written.
template <int C>
constexpr bool wave_serves(int S, int rule)
{
    return !(rule == kOptimal && S >= 8 && C >= 2 && C <= 8);
}

template <int C, int S, int BITS, int RULE = kOptimal>
void launch_orq(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    auto launch = [&](auto clip) {
        if constexpr (wave_serves<C>(S, RULE))
            launch_kernel((orq_quantize_kernel<C, S, BITS, clip.value, RULE>), dim3(nb), dim3(kWave), st, g, n, p->bucket_size,
                          p->level_iters, p->clip_factor, nb, p->seed, p->index_offset, lv, static_cast<uint32_t*>(codes));
        else
            launch_status() = hipErrorInvalidDeviceFunction;
    };
    if (p->clip_factor > 0.0f) launch(std::true_type{});
    else launch(std::false_type{});
}

template <int S, int BITS>
void launch_even_small(const float* g, size_t n, const ogq_params_t* p, float* lv, void* codes, hipStream_t st)
{
    const size_t spans = (n + 255u) / 256u;
    const dim3 grid((uint32_t)((spans + 3u) / 4u)), block(4 * kWave);
    if (p->bucket_size == 64u)
        launch_kernel((even_small_kernel<S, BITS, 4>), grid, block, st, g, n, p->clip_factor, p->seed, p->index_offset,
                           lv, static_cast<uint32_t*>(codes));
    else
        launch_kernel((even_small_kernel<S, BITS, 2>), grid, block, st, g, n, p->clip_factor, p->seed, p->index_offset,
                           lv, static_cast<uint32_t*>(codes));
}

template <int S, int BITS, int RULE>
void launch_sorted_small(const float* g, size_t n, const ogq_params_t* p, float* lv, void* codes, hipStream_t st)
{
    const size_t spans = (n + 255u) / 256u;
    const dim3 grid((uint32_t)((spans + 3u) / 4u)), block(4 * kWave);
    if (p->bucket_size == 64u)
        launch_kernel((sorted_small_kernel<S, BITS, 4, RULE>), grid, block, st, g, n, p->level_iters, p->clip_factor,
                           p->seed, p->index_offset, lv, static_cast<uint32_t*>(codes));
    else
        launch_kernel((sorted_small_kernel<S, BITS, 2, RULE>), grid, block, st, g, n, p->level_iters, p->clip_factor,
                           p->seed, p->index_offset, lv, static_cast<uint32_t*>(codes));
}

template <int C, int RULE>
void launch_paper_counts(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes,
                         hipStream_t st)
{
    if constexpr (C == 1 && (RULE == kOptimal || RULE == kLinear)) {
        // buckets of 64 and 128 elements, sorted in registers, several per wavefront
        if (p->bucket_size == 64u || p->bucket_size == 128u) {
            switch (p->bits) {
                case 2: launch_sorted_small<3, 2, RULE>(g, n, p, lv, codes, st); break;
                case 3: launch_sorted_small<5, 3, RULE>(g, n, p, lv, codes, st); break;
                default: launch_sorted_small<9, 4, RULE>(g, n, p, lv, codes, st); break;
            }
            return;
        }
    }
    if constexpr (C == 1 && RULE == kEven) {
        // buckets of 64 and 128 elements: several buckets per wavefront
        if (p->bucket_size == 64u || p->bucket_size == 128u) {
            switch (p->bits) {
                case 2: launch_even_small<3, 2>(g, n, p, lv, codes, st); break;
                case 3: launch_even_small<5, 3>(g, n, p, lv, codes, st); break;
                default: launch_even_small<9, 4>(g, n, p, lv, codes, st); break;
            }
            return;
        }
    }
    switch (p->bits) {  // 2^(bits-1) + 1 levels
        case 2: launch_orq<C, 3, 2, RULE>(g, n, p, nb, lv, codes, st); break;
        case 3: launch_orq<C, 5, 3, RULE>(g, n, p, nb, lv, codes, st); break;
        default: launch_orq<C, 9, 4, RULE>(g, n, p, nb, lv, codes, st); break;
    }
}

template <int C>
void launch_orq_levels(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes,
                       hipStream_t st)
{
    switch (p->scheme) {
        case OGQ_BINGRAD_PB:
            if constexpr (C == 1) {
                if (p->bucket_size == 64u || p->bucket_size == 128u) {
                    launch_sorted_small<2, 1, kPb>(g, n, p, lv, codes, st);
                    break;
                }
            }
            launch_orq<C, 2, 1, kPb>(g, n, p, nb, lv, codes, st);
            break;
        case OGQ_ORQ:
            if constexpr (C == 1) {
                // buckets of 64 and 128 elements, sorted in registers, several per wavefront
                if (p->bucket_size == 64u || p->bucket_size == 128u) {
                    if (p->bits == 1) launch_sorted_small<2, 1, kOptimal>(g, n, p, lv, codes, st);
                    else if (p->bits == 2) launch_sorted_small<4, 2, kOptimal>(g, n, p, lv, codes, st);
                    else launch_sorted_small<8, 3, kOptimal>(g, n, p, lv, codes, st);
                    break;
                }
            }
            switch (p->bits) {
                case 1: launch_orq<C, 2, 1>(g, n, p, nb, lv, codes, st); break;
                case 2: launch_orq<C, 4, 2>(g, n, p, nb, lv, codes, st); break;
                default: launch_orq<C, 8, 3>(g, n, p, nb, lv, codes, st); break;
            }
            break;
        case OGQ_EVEN: launch_paper_counts<C, kEven>(g, n, p, nb, lv, codes, st); break;
        case OGQ_LINEAR: launch_paper_counts<C, kLinear>(g, n, p, nb, lv, codes, st); break;
        default: launch_paper_counts<C, kOptimal>(g, n, p, nb, lv, codes, st); break;  // OGQ_ORQ_PAPER
    }
}

template <int W, int C>
constexpr bool team_serves(int S, int rule)
{
    if (W == 2) return C == 8 ? rule == kPb : S >= 8 && rule == kOptimal;
    if (W * C == 64 || W * C == 128) {
        if (C == 8) return rule == kEven || (S != 3 && rule != kPb);
        return rule == kPb || (W == 8 && S != 3 && rule != kEven);
    }
    if (W == 4 && C == 8) return S != 3 || rule == kEven;
    if (W == 4 && C == 1) return S < 8 || rule != kOptimal;
    return true;
}

template <int W, int C, int S, int BITS, int RULE = kOptimal>
void launch_orq_team(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if constexpr (team_serves<W, C>(S, RULE))
        launch_kernel((orq_team_kernel<W, C, S, BITS, RULE>), dim3(nb), dim3(W * kWave), st, g, n, p->bucket_size,
                      p->level_iters, p->clip_factor, nb, p->seed, p->index_offset, lv, static_cast<uint32_t*>(codes));
    else
        launch_status() = hipErrorInvalidDeviceFunction;
}

template <int W, int C, int RULE>
void launch_team_paper_counts(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes,
                              hipStream_t st)
{
    switch (p->bits) {  // 2^(bits-1) + 1 levels
        case 2: launch_orq_team<W, C, 3, 2, RULE>(g, n, p, nb, lv, codes, st); break;
        case 3: launch_orq_team<W, C, 5, 3, RULE>(g, n, p, nb, lv, codes, st); break;
        default: launch_orq_team<W, C, 9, 4, RULE>(g, n, p, nb, lv, codes, st); break;
    }
}

template <int W, int C>
void launch_orq_team_levels(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes,
                            hipStream_t st)
{
    switch (p->scheme) {
        case OGQ_BINGRAD_PB: launch_orq_team<W, C, 2, 1, kPb>(g, n, p, nb, lv, codes, st); break;
        case OGQ_ORQ:
            switch (p->bits) {
                case 1: launch_orq_team<W, C, 2, 1>(g, n, p, nb, lv, codes, st); break;
                case 2: launch_orq_team<W, C, 4, 2>(g, n, p, nb, lv, codes, st); break;
                default: launch_orq_team<W, C, 8, 3>(g, n, p, nb, lv, codes, st); break;
            }
            break;
        case OGQ_EVEN: launch_team_paper_counts<W, C, kEven>(g, n, p, nb, lv, codes, st); break;
        case OGQ_LINEAR: launch_team_paper_counts<W, C, kLinear>(g, n, p, nb, lv, codes, st); break;
        default: launch_team_paper_counts<W, C, kOptimal>(g, n, p, nb, lv, codes, st); break;  // OGQ_ORQ_PAPER
    }
}

}  // namespace ogq
#endif  // OGQ_ROUNDING_KERNELS_H
