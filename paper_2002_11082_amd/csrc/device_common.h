// Internal header of libogq: wave-level helpers shared by its kernel sources (gfx950, wave64).
// Everything here is inline device code or a compile-time constant; nothing is exported.
#ifndef OGQ_DEVICE_COMMON_H
#define OGQ_DEVICE_COMMON_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ogq.h"

namespace ogq {

constexpr int kWave = 64;
constexpr int kWavesPerBlock = 4;
constexpr int kBlock = kWave * kWavesPerBlock;

// ----------------------------------------------------------------------------------------------
// wave-level helpers
// ----------------------------------------------------------------------------------------------
// Cross-lane moves within a row of 16 lanes (DPP): quad_perm [1,0,3,2], quad_perm [2,3,0,1],
// row_half_mirror, row_mirror.  After the four steps of a butterfly every lane of a row holds the
// row's result; the four rows are then combined through readlane.
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x)
{
    return __uint_as_float(dpp_u32<CTRL>(__float_as_uint(x)));
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = dpp_u32<CTRL>((uint32_t)u), hi = dpp_u32<CTRL>((uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ double readlane_f64(double x, int lane)
{
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

__device__ __forceinline__ float readlane_f32(float x, int lane)
{
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), lane));
}

// v_writelane_b32 through the compiler's own intrinsic (the compiler then inserts the wait states the
// instruction needs after a VALU write of its scalar source; hand-written asm would not get them).
extern "C" __device__ uint32_t ogq_llvm_writelane(uint32_t value, uint32_t lane, uint32_t old) __asm("llvm.amdgcn.writelane.i32");

// Lane `lane` of `dst` takes the wave-uniform value `value`; the other lanes keep theirs.
__device__ __forceinline__ uint32_t writelane(uint32_t dst, uint32_t value, int lane)
{
    return ogq_llvm_writelane(value, (uint32_t)lane, dst);
}

// Wave-wide sum; the result is wave-uniform.  Four butterfly steps leave every row's sum in all of its lanes; two row
// broadcasts (DPP row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3) then add them up as (r0 + r1) + (r2 + r3)
// in the last row, from which one lane is read.
__device__ __forceinline__ double wave_sum(double x)
{
    x += dpp_f64<kDppXor1>(x);
    x += dpp_f64<kDppXor2>(x);
    x += dpp_f64<kDppHalfMirror>(x);
    x += dpp_f64<kDppMirror>(x);
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    const uint32_t lo15 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x142, 0xA, 0xF, false);
    const uint32_t hi15 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x142, 0xA, 0xF, false);
    x += __longlong_as_double((long long)(((uint64_t)hi15 << 32) | lo15));  // rows 0 and 2 add +0.0
    const uint64_t w = (uint64_t)__double_as_longlong(x);
    const uint32_t lo31 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)w, 0x143, 0xC, 0xF, false);
    const uint32_t hi31 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(w >> 32), 0x143, 0xC, 0xF, false);
    x += __longlong_as_double((long long)(((uint64_t)hi31 << 32) | lo31));
    return readlane_f64(x, 63);
}

__device__ __forceinline__ float wave_sum_f32(float x)
{
    x += dpp_f32<kDppXor1>(x);
    x += dpp_f32<kDppXor2>(x);
    x += dpp_f32<kDppHalfMirror>(x);
    x += dpp_f32<kDppMirror>(x);
    return (readlane_f32(x, 0) + readlane_f32(x, 16)) + (readlane_f32(x, 32) + readlane_f32(x, 48));
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x)
{
    x += dpp_u32<kDppXor1>(x);
    x += dpp_u32<kDppXor2>(x);
    x += dpp_u32<kDppHalfMirror>(x);
    x += dpp_u32<kDppMirror>(x);
    return (__builtin_amdgcn_readlane(x, 0) + __builtin_amdgcn_readlane(x, 16)) +
           (__builtin_amdgcn_readlane(x, 32) + __builtin_amdgcn_readlane(x, 48));
}

// Smallest and largest value of the wavefront, wave-uniform: six steps of one instruction each (the compiler makes three of a minimum across
// lanes: move, quiet, minimum; 30 instructions fewer per wavefront), the last two as in wave_sum.  Wait states: two between a write and a move of what it wrote (before the
// first step anything may have written the values), one before a lane is read.  All lanes are active.
__device__ __forceinline__ void wave_extremes(float& low, float& high)
{
#define OGQ_STEP(move) \
    "s_nop 1\n\tv_min_f32_dpp %0, %0, %0 " move "\n\tv_max_f32_dpp %1, %1, %1 " move "\n\t"
#define OGQ_ALL " row_mask:0xf bank_mask:0xf"
    asm(OGQ_STEP("quad_perm:[1,0,3,2]" OGQ_ALL) OGQ_STEP("quad_perm:[2,3,0,1]" OGQ_ALL) OGQ_STEP("row_half_mirror" OGQ_ALL)
            OGQ_STEP("row_mirror" OGQ_ALL) OGQ_STEP("row_bcast:15 row_mask:0xa bank_mask:0xf") OGQ_STEP("row_bcast:31 row_mask:0xc bank_mask:0xf") "s_nop 1"
        : "+v"(low), "+v"(high));
#undef OGQ_ALL
#undef OGQ_STEP
    low = readlane_f32(low, 63);
    high = readlane_f32(high, 63);
}

__device__ __forceinline__ float wave_max(float x)
{
    x = fmaxf(x, dpp_f32<kDppXor1>(x));
    x = fmaxf(x, dpp_f32<kDppXor2>(x));
    x = fmaxf(x, dpp_f32<kDppHalfMirror>(x));
    x = fmaxf(x, dpp_f32<kDppMirror>(x));
    return fmaxf(fmaxf(readlane_f32(x, 0), readlane_f32(x, 16)), fmaxf(readlane_f32(x, 32), readlane_f32(x, 48)));
}

constexpr int kDppRor8 = 0x128;   // rotate by 8 inside a row of 16 lanes: partner lane ^ 8
constexpr int kDppRowShl4 = 0x104;  // lane i takes lane i + 4 of its row
constexpr int kDppRowShr4 = 0x114;  // lane i takes lane i - 4 of its row

// Value held by lane (lane ^ DIST).
template <int DIST>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x, uint32_t lane)
{
    if constexpr (DIST == 1) {
        return dpp_u32<kDppXor1>(x);
    } else if constexpr (DIST == 2) {
        return dpp_u32<kDppXor2>(x);
    } else if constexpr (DIST == 4) {
        // banks (groups of 4 lanes) 0 and 2 of every row take the lane 4 above, banks 1 and 3 the lane 4 below
        int y = __builtin_amdgcn_update_dpp((int)x, (int)x, kDppRowShl4, 0xF, 0x5, false);
        y = __builtin_amdgcn_update_dpp(y, (int)x, kDppRowShr4, 0xF, 0xA, false);
        return (uint32_t)y;
    } else if constexpr (DIST == 8) {
        return dpp_u32<kDppRor8>(x);
    } else if constexpr (DIST == 16) {
        // rows (0,1) and (2,3) trade places
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (lane & 16u) ? r[0] : r[1];
    } else {
        // the two halves of the wave trade places
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return (lane & 32u) ? r[0] : r[1];
    }
}

// 8 x 8 transpose of nibbles inside every group of 8 lanes: lane i's nibble c and lane c's nibble i trade places.  Three
// butterfly steps; those that move whole bytes are one cross-lane move and one byte permute.
struct NibbleTranspose {
    uint32_t swap16, swap8;  // byte selectors of the steps over lane bits 2 and 1
    uint32_t take, turn;     // the step over lane bit 0: nibbles taken from the partner, right rotation that places them
};

__device__ __forceinline__ NibbleTranspose nibble_transpose_setup(uint32_t lane)
{
    // the lower lane of a pair keeps its low blocks and takes the partner's low blocks as its high blocks, the upper lane
    // keeps its high blocks and takes the partner's high blocks as its low blocks (bytes 0 .. 3: own, 4 .. 7: partner's)
    NibbleTranspose t;
    t.swap16 = (lane & 4u) ? 0x03020706u : 0x05040100u;
    t.swap8 = (lane & 2u) ? 0x03070105u : 0x06020400u;
    t.take = (lane & 1u) ? 0x0F0F0F0Fu : 0xF0F0F0F0u;
    t.turn = (lane & 1u) ? 4u : 28u;
    return t;
}

__device__ __forceinline__ uint32_t nibble_transpose(uint32_t x, const NibbleTranspose& t, uint32_t lane)
{
    x = __builtin_amdgcn_perm(lane_xor<4>(x, lane), x, t.swap16);
    x = __builtin_amdgcn_perm(lane_xor<2>(x, lane), x, t.swap8);
    const uint32_t y = lane_xor<1>(x, lane);
    // take ? turned : x, bit by bit, in one instruction (v_bitop3_b32, truth table 0xCA)
    return __builtin_amdgcn_bitop3_b32(t.take, __builtin_amdgcn_alignbit(y, y, t.turn), x, 0xCA);
}

// v within [-limit, limit], in one instruction (v_med3_f32).  limit = NaN (a bucket that is not finite): v as it is.
__device__ __forceinline__ float clipped(float v, float limit) { return __builtin_amdgcn_fmed3f(v, -limit, limit); }

// Variance times length of a bucket from its sum and its sum of squares, which fp64 fma adds without rounding a product (48 bits).
// `cancels`: the square of the bucket's mean is more than an eighth of the mean of its squares, so that the difference would lose more than a part
// of a bit; such a bucket takes the sum of the squares about its mean, and most of those that are not finite (with an infinity among its values the result
// is NaN either way).
__device__ __forceinline__ double squares_about_mean(double sum, double squares, double len, bool& cancels)
{
    const double mean = sum / len;
    cancels = !(sum * mean <= 0.125 * squares);
    return __builtin_fma(-sum, mean, squares);
}

// Gradient clipping of a register-resident bucket (Section 5): v <- sign(v) * min(|v|, c * sigma) with
// sigma^2 the population variance about the bucket mean, in fp64.  valid(j) tells whether
// register j of this lane holds a bucket element; bucket_sums(x, y) adds x and y over all lanes that hold the bucket.  MEET: it has
// barriers at which wavefronts of other buckets wait too, so that all call it equally often.  Returns the threshold.  (One pass and one
// reduction in place of two, and v_med3 in place of three instructions: nine levels, buckets of 512, 25.6 M values 68.0 -> 65.1 us.)
template <int N, bool MEET = false, class ValidFn, class SumsFn>
__device__ __forceinline__ float clip_in_registers(float (&v)[N], uint32_t len, float c, ValidFn valid, SumsFn bucket_sums)
{
    double about_mean;
    if constexpr (N <= 2) {  // (a second pass over one or two values costs less than the test of the first: BinGrad-b, 11719 buckets of 128, 7.6 us and 7.9)
        double sum = 0.0, unused = 0.0;
#pragma unroll
        for (int j = 0; j < N; ++j) sum += valid(j) ? (double)v[j] : 0.0;
        bucket_sums(sum, unused);
        const double mean = sum / (double)len;
        about_mean = 0.0;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const double dv = (double)v[j] - mean;
            about_mean += valid(j) ? dv * dv : 0.0;
        }
        bucket_sums(about_mean, unused);
    } else {
        double sum = 0.0, squares = 0.0;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const double x = valid(j) ? (double)v[j] : 0.0;
            sum += x;
            squares = __builtin_fma(x, x, squares);
        }
        bucket_sums(sum, squares);
        bool cancels;
        about_mean = squares_about_mean(sum, squares, (double)len, cancels);
        double part = 0.0, unused = 0.0;
        const bool again = __ballot(cancels) != 0;  // (every wavefront of a bucket, or none: they hold the same sums)
        if (__builtin_expect(again, 0)) {
            const double mean = sum / (double)len;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                // converted again: fp64 copies of 32 values kept from the first pass would not fit the registers
                asm volatile("" : "+v"(v[j]));
                const double dv = (double)v[j] - mean;
                part += valid(j) ? dv * dv : 0.0;
            }
        }
        if (MEET || again) bucket_sums(part, unused);
        about_mean = cancels ? part : about_mean;
    }
    const float limit = (float)((double)c * sqrt(about_mean / (double)len));
#pragma unroll
    for (int j = 0; j < N; ++j) v[j] = clipped(v[j], limit);
    return limit;
}

template <int N, class ValidFn>
__device__ __forceinline__ float clip_in_registers(float (&v)[N], uint32_t len, float c, ValidFn valid)
{
    return clip_in_registers<N>(v, len, c, valid, [](double& x, double& y) {
        x = wave_sum(x);
        y = wave_sum(y);
    });
}

__device__ __forceinline__ uint32_t uniform_u32(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ __forceinline__ float uniform_f32(float x)
{
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

__device__ __forceinline__ double uniform_f64(double x)
{
    uint64_t u = (uint64_t)__double_as_longlong(x);
    uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
    uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// ----------------------------------------------------------------------------------------------
// A bucket is held by one wavefront, or by the W wavefronts of a workgroup: the Team types say how a
// wave-wide result becomes a bucket-wide one.
// ----------------------------------------------------------------------------------------------
struct OneWave {
    static constexpr int kSize = 1;
    __device__ __forceinline__ double sum(double x) { return x; }
    __device__ __forceinline__ void sums(double&, double&) {}
    __device__ __forceinline__ void sum_and_max(double&, float&) {}
    __device__ __forceinline__ void sum_and_count(double&, uint32_t&) {}
};

// All wavefronts of the team call every combine in the same order (their control flow depends on combined
// values only).  Two alternating LDS slots are enough: a wavefront that writes a slot for the second time has
// passed the barrier in between, which the others reach only after they have read the first value.
struct TeamSlot {
    double sum;
    uint32_t a, b;
};

template <int W>
struct WaveTeam {
    static constexpr int kSize = W;
    TeamSlot (*slots)[W];  // [2][W] in LDS: [call parity][wavefront]
    uint32_t wave;
    uint32_t calls;
    __device__ __forceinline__ const TeamSlot* exchange(double sum, uint32_t a, uint32_t b)
    {
        TeamSlot* slot = slots[calls & 1u];
        ++calls;
        if ((threadIdx.x & 63u) == 0) {
            slot[wave].sum = sum;
            slot[wave].a = a;
            slot[wave].b = b;
        }
        __syncthreads();
        return slot;
    }
    __device__ __forceinline__ double sum(double x)
    {
        const TeamSlot* s = exchange(x, 0u, 0u);
        double r = s[0].sum;
#pragma unroll
        for (int w = 1; w < W; ++w) r += s[w].sum;
        return r;
    }
    __device__ __forceinline__ void sums(double& x, double& y)
    {
        const uint64_t u = (uint64_t)__double_as_longlong(y);
        const TeamSlot* s = exchange(x, (uint32_t)u, (uint32_t)(u >> 32));
        auto other = [](const TeamSlot& t) { return __longlong_as_double((long long)((uint64_t)t.b << 32 | t.a)); };
        x = s[0].sum;
        y = other(s[0]);
#pragma unroll
        for (int w = 1; w < W; ++w) {
            x += s[w].sum;
            y += other(s[w]);
        }
    }
    __device__ __forceinline__ void sum_and_max(double& x, float& m)
    {
        const TeamSlot* s = exchange(x, __float_as_uint(m), 0u);
        x = s[0].sum;
        m = __uint_as_float(s[0].a);
#pragma unroll
        for (int w = 1; w < W; ++w) {
            x += s[w].sum;
            m = fmaxf(m, __uint_as_float(s[w].a));
        }
    }
    __device__ __forceinline__ void sum_and_count(double& x, uint32_t& c)
    {
        const TeamSlot* s = exchange(x, c, 0u);
        x = s[0].sum;
        c = s[0].a;
#pragma unroll
        for (int w = 1; w < W; ++w) {
            x += s[w].sum;
            c += s[w].a;
        }
    }
};

}  // namespace ogq
#endif  // OGQ_DEVICE_COMMON_H
