// libogq, decode + average kernel (server step of Algorithm 2 of arXiv 2002.11082) and the bandwidth probes,
// for MI355X (gfx950).
#include <type_traits>

#include "device_common.h"
#include "launch.h"

namespace ogq {

// ----------------------------------------------------------------------------------------------
// Decode + average.  One wavefront decodes a span of up to 16 packed word groups (1024 elements); lane l owns
// element 64*j + l of word group j.  For bucket sizes with a fixed place in a span (64 .. 512 and multiples of 1024), and
// there for a single worker or buckets below 512 elements: everything else takes dequantize_joint_kernel.  Complete
// spans turn the code bits into per-lane level indices and look the levels up in LDS (below); the ragged last span uses
// the packed words directly as the lane masks of a tree of selects.
// ----------------------------------------------------------------------------------------------
// N: the most workers it holds.  It travels as a kernel argument, and a launch with 1 KB of arguments takes 0.6 us longer
// on the host than one with 128 bytes: launches of one, up to eight and more workers have instantiations of their own.
template <int N>
struct WorkerPtrs {
    const uint64_t* codes[N];
    const float* levels[N];
};
constexpr int kFewWorkers = 8;

constexpr int kSpanWords = 16;  // one wavefront decodes 16 packed word groups = 1024 elements

__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Level selected by the packed words of one 64-element group: the words are the lane masks of the
// selects.  S = 2^BITS levels: a full binary tree; S = 2^(BITS-1) + 1 levels (the paper's counts):
// the top bit alone means the last level.
template <int BITS>
__device__ __forceinline__ float select_tree(const bool (&bit)[4], const float* lv)
{
    if constexpr (BITS == 0) {
        return lv[0];
    } else {
        const float lo = select_tree<BITS - 1>(bit, lv);
        const float hi = select_tree<BITS - 1>(bit, lv + (1 << (BITS - 1)));
        return bit[BITS - 1] ? hi : lo;
    }
}

template <int BITS, int S>
__device__ __forceinline__ float select_level(const uint64_t* __restrict__ w, const float (&lv)[S])
{
    bool bit[4] = {false, false, false, false};
#pragma unroll
    for (int p = 0; p < BITS; ++p) bit[p] = __builtin_amdgcn_inverse_ballot_w64(w[p]);
    if constexpr (S == (1 << BITS)) {
        return select_tree<BITS>(bit, lv);
    } else {
        static_assert(S == (1 << (BITS - 1)) + 1, "level count");
        const float low = select_tree<BITS - 1>(bit, lv);
        return bit[BITS - 1] ? lv[S - 1] : low;
    }
}

// Loads one bucket's level table (wave-uniform address, scalar loads) into vector registers: the
// selects take two vector sources and the packed word as their lane mask.
template <int S>
__device__ __forceinline__ void load_levels(const float* __restrict__ table, float (&lv)[S])
{
    float s[S];
#pragma unroll
    for (int k = 0; k < S; ++k) s[k] = table[k];
#pragma unroll
    for (int k = 0; k < S; ++k) asm("v_mov_b32 %0, %1" : "=v"(lv[k]) : "s"(s[k]));
}

// ----------------------------------------------------------------------------------------------
// The span's code bits, turned so that every lane holds the bits of its own elements.  A span's code words are
// 16 * BITS rows of 64 bits (row = word group * BITS + bit plane, one bit per element of the group).  Lane 32 h + r
// loads the half h (32 elements) of rows r, r + 32, ...; a 32 x 32 bit-matrix transpose inside each half of the
// wavefront (five butterfly steps: the partner lane's word, rotated, replaces half of the bits) then leaves, in lane
// 32 h + b, bit `row` of the result = code bit of element 32 h + b of that row's group: the level index of group j
// sits at bits BITS j .. BITS j + BITS - 1 and indexes the bucket's level table in LDS directly.
// ----------------------------------------------------------------------------------------------
struct BitTranspose {
    uint32_t take[5];  // bits a lane takes from its partner at lane distance 16, 8, 4, 2, 1
    uint32_t turn[5];  // right rotation that brings the partner's bits into place
};

__device__ __forceinline__ BitTranspose bit_transpose_setup(uint32_t lane)
{
    BitTranspose t;
    constexpr uint32_t kLow[5] = {0x0000FFFFu, 0x00FF00FFu, 0x0F0F0F0Fu, 0x33333333u, 0x55555555u};
#pragma unroll
    for (int s = 0; s < 5; ++s) {
        const uint32_t j = 16u >> s;
        const bool upper = (lane & j) != 0u;
        // the lower lane of a pair keeps its low blocks and takes the partner's low blocks as its high blocks; the upper
        // lane keeps its high blocks and takes the partner's high blocks as its low blocks
        t.take[s] = upper ? kLow[s] : kLow[s] << j;
        t.turn[s] = upper ? j : 32u - j;
    }
    return t;
}

template <int DIST, int STEP>
__device__ __forceinline__ uint32_t bit_transpose_step(uint32_t x, const BitTranspose& t, uint32_t lane)
{
    const uint32_t y = lane_xor<DIST>(x, lane);
    const uint32_t turned = __builtin_amdgcn_alignbit(y, y, t.turn[STEP]);
    // take ? turned : x, bit by bit, in one instruction (v_bitop3_b32, truth table 0xCA)
    return __builtin_amdgcn_bitop3_b32(t.take[STEP], turned, x, 0xCA);
}

__device__ __forceinline__ uint32_t bit_transpose(uint32_t x, const BitTranspose& t, uint32_t lane)
{
    x = bit_transpose_step<16, 0>(x, t, lane);
    x = bit_transpose_step<8, 1>(x, t, lane);
    x = bit_transpose_step<4, 2>(x, t, lane);
    x = bit_transpose_step<2, 3>(x, t, lane);
    return bit_transpose_step<1, 4>(x, t, lane);
}

// Level index of word group J from the turned code bits (R registers of 32 rows each).
template <int BITS, int J, int R>
__device__ __forceinline__ uint32_t level_index(const uint32_t (&turned)[R])
{
    constexpr int kFirst = BITS * J, kReg = kFirst / 32, kShift = kFirst % 32;
    uint32_t index;
    if constexpr (kShift + BITS <= 32) {
        index = __builtin_amdgcn_ubfe(turned[kReg], (uint32_t)kShift, (uint32_t)BITS);  // one v_bfe_u32
    } else {
        index = __builtin_amdgcn_alignbit(turned[kReg + 1], turned[kReg], (uint32_t)kShift) & ((1u << BITS) - 1u);
    }
    // (kept as it is: folded into the address arithmetic, the extraction turns into a shift, a mask and an addition
    // instead of this bit-field extract and one shift-and-add)
    asm("" : "+v"(index));
    return index;
}

// Runs f(J, index of word group J) for the 16 word groups of a span; an index has BITS bits.
template <int BITS, int J, int R, class F>
__device__ __forceinline__ void for_each_group(const uint32_t (&turned)[R], F&& f)
{
    if constexpr (J < kSpanWords) {
        f(std::integral_constant<int, J>{}, level_index<BITS, J>(turned));
        for_each_group<BITS, J + 1>(turned, f);
    }
}

// WPB = packed word groups per bucket: 16 = the span lies in one bucket (bucket_size is a multiple of 1024; its index is
// word0 / words_per_bucket), 1, 2, 4 or 8 = bucket_size 64 .. 512, the span holds 16 / WPB buckets whose level tables
// are consecutive in memory.  Each table is fetched once per span and worker.
// MOST: what the worker list holds.  1: the launch has a single worker (without the fp64 sums of the general case the
// kernel needs half the registers, and twice the wavefronts are in flight to hide the first trip to HBM).
template <int BITS, int S, int WPB, int MOST>
__global__ __launch_bounds__(kBlock) void dequantize_average_kernel(WorkerPtrs<MOST> ptrs, uint32_t num_workers, size_t n,
                                                                    uint32_t words_per_bucket, uint32_t total_words,
                                                                    double inv_workers, float* __restrict__ out)
{
    constexpr bool ONE = MOST == 1;
    const uint32_t span = blockIdx.x * kWavesPerBlock + uniform_u32(threadIdx.x >> 6);
    const uint32_t word0 = span * kSpanWords;
    if (word0 >= total_words) return;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t rest = total_words - word0;
    const uint32_t n_words = rest < (uint32_t)kSpanWords ? rest : (uint32_t)kSpanWords;
    // every element of the span exists: no per-word or per-element bounds tests
    const bool whole = n_words == (uint32_t)kSpanWords && ((size_t)word0 + kSpanWords) * 64 <= n;

    double acc[kSpanWords];
#pragma unroll
    for (int j = 0; j < kSpanWords; ++j) acc[j] = 0.0;

    if (whole) {
        // Every element of the span exists and its buckets lie at fixed places: the span's code words and level
        // tables are fetched with vector loads (one dword per lane and register), for several workers at once so
        // that their trips to HBM overlap.  The code bits are turned into per-lane level indices (bit_transpose), the
        // level tables go to a table in LDS that belongs to this wavefront, and an element's level is one LDS read.
        // (Scalar loads, which would deliver the words as lane masks for a select tree, keep too few bytes in flight
        // per wavefront once the streams come from HBM instead of the last-level cache; moving vector-loaded words
        // to scalar registers costs two v_readlane per word.)
        constexpr int kTables = kSpanWords / WPB;
        const BitTranspose turn = bit_transpose_setup(lane);
        const uint32_t half = lane >> 5, row = lane & 31u;
        const uint32_t first_bucket = WPB == kSpanWords ? word0 / words_per_bucket : word0 / (uint32_t)WPB;
        const uint32_t wave = uniform_u32(threadIdx.x >> 6);
        {
            // One worker per look-up: fp32 level tables in LDS.  A single worker's average is its level itself.
            constexpr int R = (kSpanWords * BITS + 31) / 32;  // registers for the 16 * BITS rows of code bits
            constexpr int LR = (kTables * S + 63) / 64;       // registers for the kTables * S level values
            constexpr uint32_t BATCH = R + LR > 2 ? 4 : 8;    // workers whose loads are in flight together
            __shared__ float level_tables[kWavesPerBlock][BATCH * kTables * S];
            float* my_tables = level_tables[wave];
            constexpr bool one_worker = ONE;
            for (uint32_t w0 = 0; w0 < num_workers; w0 += BATCH) {
                uint32_t code_reg[BATCH][R];
                float level_reg[BATCH][LR];
#pragma unroll
                for (uint32_t b = 0; b < BATCH; ++b) {
#pragma unroll
                    for (int k = 0; k < R; ++k) code_reg[b][k] = 0u;
#pragma unroll
                    for (int k = 0; k < LR; ++k) level_reg[b][k] = 0.0f;
                    if (w0 + b < num_workers) {
                        const uint32_t* c32 = reinterpret_cast<const uint32_t*>(ptrs.codes[w0 + b] + (size_t)word0 * BITS);
                        const float* tables = ptrs.levels[w0 + b] + (size_t)first_bucket * S;
#pragma unroll
                        for (int k = 0; k < R; ++k) {
                            const uint32_t r = 32u * k + row;  // row of code bits this lane fetches its half of
                            if (r < (uint32_t)(kSpanWords * BITS)) code_reg[b][k] = c32[2u * r + half];
                        }
#pragma unroll
                        for (int k = 0; k < LR; ++k) {
                            const uint32_t i = 64u * k + lane;
                            if (i < (uint32_t)(kTables * S)) level_reg[b][k] = tables[i];
                        }
                    }
                }
                wave_lds_fence();  // the reads of the batch before are done
#pragma unroll
                for (uint32_t b = 0; b < BATCH; ++b) {
#pragma unroll
                    for (int k = 0; k < LR; ++k) {
                        const uint32_t i = 64u * k + lane;
                        if (i < (uint32_t)(kTables * S)) my_tables[b * (kTables * S) + i] = level_reg[b][k];
                    }
                }
                wave_lds_fence();
#pragma unroll
                for (uint32_t b = 0; b < BATCH; ++b) {
                    if (w0 + b < num_workers) {
                        uint32_t turned[R];
#pragma unroll
                        for (int k = 0; k < R; ++k) turned[k] = bit_transpose(code_reg[b][k], turn, lane);
                        const float* table = my_tables + b * (kTables * S);
                        if (one_worker) {
                            float* __restrict__ o1 = out + (size_t)word0 * 64 + lane;
                            for_each_group<BITS, 0>(turned, [&](auto j, uint32_t index) {
                                // written once, never re-read here
                                __builtin_nontemporal_store(table[(decltype(j)::value / WPB) * S + index], o1 + 64 * decltype(j)::value);
                            });
                            return;
                        }
                        for_each_group<BITS, 0>(turned, [&](auto j, uint32_t index) {
                            acc[decltype(j)::value] += (double)table[(decltype(j)::value / WPB) * S + index];
                        });
                    }
                }
            }
        }
    } else  // the ragged end of the gradient: scalar loads, word by word
    for (uint32_t w = 0; w < num_workers; ++w) {
        const uint64_t* __restrict__ cw = ptrs.codes[w] + (size_t)word0 * BITS;
        constexpr int kTables = kSpanWords / WPB;
        const uint32_t first_bucket = WPB == kSpanWords ? word0 / words_per_bucket : word0 / (uint32_t)WPB;
        const float* __restrict__ first_table = ptrs.levels[w] + (size_t)first_bucket * S;
#pragma unroll
        for (int t = 0; t < kTables; ++t)
            if ((uint32_t)(t * WPB) < n_words) {  // a bucket past the end has no table
                float lv[S];
                load_levels<S>(first_table + t * S, lv);
#pragma unroll
                for (int j = t * WPB; j < (t + 1) * WPB; ++j)
                    if ((uint32_t)j < n_words) acc[j] += (double)select_level<BITS, S>(cw + j * BITS, lv);
            }
    }
    float* __restrict__ o = out + (size_t)word0 * 64 + lane;
    if (whole) {
#pragma unroll
        for (int j = 0; j < kSpanWords; ++j)
            __builtin_nontemporal_store((float)(acc[j] * inv_workers), o + 64 * j);  // written once, never re-read here
    } else {
        const size_t first = (size_t)word0 * 64 + lane;
#pragma unroll
        for (int j = 0; j < kSpanWords; ++j)
            if ((uint32_t)j < n_words && first + 64u * j < n)
                __builtin_nontemporal_store((float)(acc[j] * inv_workers), o + 64 * j);
    }
}

// ----------------------------------------------------------------------------------------------
// Decode + average with table look-ups for K workers at once: K = 8 with one-bit codes, 4 with two, 2 with three and four.
//
// One wavefront per span of 1024 elements; chunk c, lane l: elements 256c + 4l + {0..3}, so that the averages leave in four
// 16-byte stores per lane.  What bounds it: instruction issue and latency (at eight two-bit workers 540 instructions per
// span with the 32 x 32 transposes and staged rows of dequantize_average_kernel, 82 us for 61.1 M elements against 57 us of
// HBM time; here 370 and 68 us), so the code bits reach their elements in few steps:
//   - A worker's words of the span are 64 BITS dwords (a half word of one plane each).  Lane 8h + j fetches half word h of
//     column j; a column is a chunk and a plane (from two bits on), or a chunk and one of two workers (one bit).
//   - A nibble transpose among 8 lanes (8 instructions) leaves in nibble j of every lane the bits of its own four
//     elements in column j.
//   - One and two bits: four such registers (four workers, or pairs of them) trade the worker bits against the element
//     bits of their nibbles (a 4 x 4 bit transpose, 16 instructions): byte c of register k is then the joint index of
//     the K workers for element k of chunk c.  Three and four bits: plane and element trade places inside each 16 bits,
//     and the nibbles of two workers are interleaved into bytes.
//   - The index looks up the sum of the K workers' levels, tabulated in LDS for all 256 combinations (fp64).  With at most
//     K workers the table holds the averages themselves, rounded to fp32, and one look-up per element is all.
// A span touches at most BUCKETS buckets: one if the bucket size is a multiple of 1024, two from 1024 elements on or with
// 512, three from 512 on, four from 320 on, six with 192.  Each has its own table, 2 KB per wavefront with fp64 sums; the
// LDS limits the wavefronts of a CU (room for seven tables from 192 to 448 elements: two workgroups of fp64 tables; with
// six three, with four four.  25.6 M values, eight two-bit workers: 192 elements 54.7 -> 43.2 us, 320 48.0 -> 32.5, 448
// 48.1 -> 31.6.  One-bit codes of eight workers, whose tables are fp32, 6.4 M: 8.3 -> 7.9, 25.6 M: 22.3 -> 22.7).
// ----------------------------------------------------------------------------------------------
constexpr uint32_t kJointEntries = 256;

// low & mask | (high & mask) << SHIFT, and low >> SHIFT & mask | high & ~mask: exchanges bit SHIFT of the position inside a
// register with the choice of the register.
template <int SHIFT>
__device__ __forceinline__ void exchange_bits(uint32_t& low, uint32_t& high, uint32_t mask)
{
    const uint32_t a = __builtin_amdgcn_bitop3_b32(mask, low, high << SHIFT, 0xCA);  // mask ? low : high << SHIFT
    const uint32_t b = __builtin_amdgcn_bitop3_b32(mask, low >> SHIFT, high, 0xCA);
    low = a;
    high = b;
}

// Exchanges the bits of a position whose bits LOW and HIGH differ: bit LOW of the position trades places with bit HIGH.
template <int LOW, int HIGH>
__device__ __forceinline__ uint32_t exchange_positions(uint32_t x)
{
    constexpr int kShift = (1 << HIGH) - (1 << LOW);
    constexpr uint32_t kFrom = LOW == 0 ? 0x0A0A0A0Au : 0x00CC00CCu;  // positions with bit LOW set and bit HIGH clear
    static_assert((LOW == 0 && HIGH == 2) || (LOW == 1 && HIGH == 3), "masks of these two");
    const uint32_t differ = (x ^ (x >> kShift)) & kFrom;
    return x ^ differ ^ (differ << kShift);
}

// LAST: all workers are in one look-up (num_workers <= K).
template <int BITS, int S, uint32_t BUCKETS, int MOST, bool LAST>
__global__ __launch_bounds__(kBlock) void dequantize_joint_kernel(WorkerPtrs<MOST> ptrs, uint32_t num_workers, size_t n,
                                                                  uint32_t words_per_bucket, uint32_t total_words,
                                                                  double inv_workers, float* __restrict__ out)
{
    constexpr bool NIBBLES = BITS > 2;   // an element's index is a nibble per worker
    constexpr uint32_t K = NIBBLES ? 2u : 8u / BITS;  // workers per look-up
    constexpr int GROUPS = LAST ? 1 : 2; // look-ups whose loads are in flight together
    using Entry = typename std::conditional<LAST, float, double>::type;
    __shared__ Entry tables[kWavesPerBlock][BUCKETS][kJointEntries];
    __shared__ float raw_levels[kWavesPerBlock][GROUPS][K][BUCKETS * S];
    const uint32_t wave = uniform_u32(threadIdx.x >> 6);
    const uint32_t span = blockIdx.x * kWavesPerBlock + wave;
    const uint32_t word0 = span * kSpanWords;
    if (word0 >= total_words) return;
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t words = total_words - word0 < (uint32_t)kSpanWords ? total_words - word0 : (uint32_t)kSpanWords;
    const uint32_t first_bucket = word0 / words_per_bucket;
    // The bucket of a word of the span, counted from the first one: up to three buckets by the words with which the second
    // and the third begin, for more (of 3 to 7 words) by a product with the reciprocal (exact: the words counted stay below 22).
    const uint32_t skipped = word0 - first_bucket * words_per_bucket;
    const uint32_t second = words_per_bucket - skipped, third = second + words_per_bucket;
    const uint32_t reciprocal = BUCKETS > 3u ? 65536u / words_per_bucket + 1u : 0u;
    auto bucket_of = [&](uint32_t word) {
        if constexpr (BUCKETS == 1u) return 0u;
        else if constexpr (BUCKETS <= 3u) return (word >= second ? 1u : 0u) + (BUCKETS > 2u && word >= third ? 1u : 0u);
        else return ((skipped + word) * reciprocal) >> 16;
    };
    const uint32_t buckets = bucket_of(words - 1u) + 1u;

    // lane 8 h + j fetches half word h of column j (of chunk c: word group 4 c + h / 2)
    const uint32_t column = lane & 7u, half = (lane >> 3) & 1u;
    const uint32_t group = 4u * (column >> (NIBBLES ? 2 : 1)) + (lane >> 4);
    const uint32_t plane = BITS == 1 ? 0u : column & (NIBBLES ? 3u : 1u);
    const uint32_t dword = (group * (uint32_t)BITS + plane) * 2u + half;
    const bool has_plane = BITS != 3 || plane < 3u;
    const NibbleTranspose transpose = nibble_transpose_setup(lane);
    constexpr uint32_t kMask4 = 0x0F0F0F0Fu, kMask2 = 0x33333333u, kMask1 = 0x55555555u;

    double acc[LAST ? 1 : 4][4];
    float average[4][4];
    if constexpr (!LAST) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[c][k] = 0.0;
    }
    for (uint32_t w0 = 0; w0 < num_workers; w0 += GROUPS * K) {
        uint32_t bits[GROUPS][4];
        float level[GROUPS][K];  // levels of the look-up's worker i: lane b S + s holds level s of bucket b
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) {
            const uint32_t first = w0 + q * K;
#pragma unroll
            for (uint32_t i = 0; i < 4u; ++i) {
                bits[q][i] = 0u;  // a worker that does not exist: index 0 of levels 0
                const uint32_t w = BITS == 1 ? first + 2u * i : NIBBLES ? first + i / 2u : first + i;
                const uint32_t later = NIBBLES ? 8u * (i & 1u) : 0u;  // a worker's second register: chunks 2 and 3
                if (w < num_workers) {  // (uniform)
                    const uint32_t* from = reinterpret_cast<const uint32_t*>(ptrs.codes[w] + (size_t)word0 * BITS);
                    bool mine = has_plane && later + group < words;
                    if constexpr (BITS == 1) {
                        const bool other = (column & 1u) != 0u;  // odd columns: the pair's second worker
                        const bool pair = w + 1u < num_workers;
                        const uint32_t* second_from = reinterpret_cast<const uint32_t*>(ptrs.codes[pair ? w + 1u : w] + (size_t)word0);
                        from = other ? second_from : from;
                        mine = mine && (pair || !other);
                    }
                    if (mine) bits[q][i] = from[dword + later * (uint32_t)(2 * BITS)];
                }
            }
#pragma unroll
            for (uint32_t i = 0; i < K; ++i) {
                level[q][i] = 0.0f;
                if (first + i < num_workers && lane < buckets * (uint32_t)S)
                    level[q][i] = ptrs.levels[first + i][(size_t)first_bucket * S + lane];
            }
        }
        wave_lds_fence();  // the reads of the round before are done
#pragma unroll
        for (int q = 0; q < GROUPS; ++q)
#pragma unroll
            for (uint32_t i = 0; i < K; ++i)
                if (lane < BUCKETS * (uint32_t)S) raw_levels[wave][q][i][lane] = level[q][i];
        // byte offset of the table of every chunk's bucket (the lane's four elements of a chunk share a word group)
        uint32_t table_at[4];
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) {
            table_at[c] = bucket_of(4u * c + (lane >> 4)) * (uint32_t)(kJointEntries * sizeof(Entry));
        }
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) {
            if (q > 0 && w0 + q * K >= num_workers) continue;  // (uniform) no such look-up
            wave_lds_fence();  // the levels are there, the look-ups before are done
            // Tables: entry lane + 64 t.  An index holds, from bit 0 on, the workers' lower code bits and then their upper
            // ones (two bits), the even and then the odd workers' bits (one bit), or the first and then the second
            // worker's index (three, four); its two top bits are those of t.
            for (uint32_t b = 0; b < buckets; ++b) {
                auto lv = [&](uint32_t i, uint32_t index) { return (double)raw_levels[wave][q][i][b * (uint32_t)S + index]; };
                auto bit = [&](uint32_t position) { return (lane >> position) & 1u; };
                double fixed, x[2], y[2];  // what the lane decides, and the contributions of the two top bits
                if constexpr (NIBBLES) {
                    auto at = [&](uint32_t i, uint32_t index) { return lv(i, index < (uint32_t)S ? index : (uint32_t)(S - 1)); };
                    const double first_worker = at(0u, lane & 15u);
#pragma unroll
                    for (uint32_t t = 0; t < 4u; ++t) {
                        const double sum = first_worker + at(1u, (lane >> 4) + 4u * t);
                        tables[wave][b][lane + 64u * t] = (Entry)(LAST ? sum * inv_workers : sum);
                    }
                    continue;
                } else if constexpr (BITS == 2) {
                    auto at = [&](uint32_t i, uint32_t index) { return lv(i, index < (uint32_t)S ? index : (uint32_t)(S - 1)); };
                    fixed = at(0u, 2u * bit(4) + bit(0)) + at(1u, 2u * bit(5) + bit(1));
#pragma unroll
                    for (uint32_t u = 0; u < 2u; ++u) {
                        x[u] = at(2u, 2u * u + bit(2));
                        y[u] = at(3u, 2u * u + bit(3));
                    }
                } else {
                    fixed = ((lv(0, bit(0)) + lv(2, bit(1))) + (lv(4, bit(2)) + lv(6, bit(3)))) + (lv(1, bit(4)) + lv(3, bit(5)));
#pragma unroll
                    for (uint32_t u = 0; u < 2u; ++u) {
                        x[u] = lv(5, u);
                        y[u] = lv(7, u);
                    }
                }
#pragma unroll
                for (uint32_t t = 0; t < 4u; ++t) {
                    const double sum = (fixed + x[t & 1u]) + y[t >> 1];
                    tables[wave][b][lane + 64u * t] = (Entry)(LAST ? sum * inv_workers : sum);
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) bits[q][i] = nibble_transpose(bits[q][i], transpose, lane);
            if constexpr (NIBBLES) {
#pragma unroll
                for (int i = 0; i < 4; ++i) bits[q][i] = exchange_positions<1, 3>(exchange_positions<0, 2>(bits[q][i]));
                exchange_bits<4>(bits[q][0], bits[q][2], kMask4);
                exchange_bits<4>(bits[q][1], bits[q][3], kMask4);
            } else {
                exchange_bits<2>(bits[q][0], bits[q][2], kMask2);
                exchange_bits<2>(bits[q][1], bits[q][3], kMask2);
                exchange_bits<1>(bits[q][0], bits[q][1], kMask1);
                exchange_bits<1>(bits[q][2], bits[q][3], kMask1);
            }
            wave_lds_fence();
            const char* base = reinterpret_cast<const char*>(&tables[wave][0][0]);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    // (nibbles: registers 0 and 1 hold elements 0 and 2 of chunks 0, 1 and 2, 3, registers 2 and 3 the others)
                    const uint32_t reg = NIBBLES ? bits[q][2 * (k & 1) + c / 2] : bits[q][k];
                    const uint32_t index = __builtin_amdgcn_ubfe(reg, NIBBLES ? 16u * (c & 1) + 8u * (k / 2) : 8u * c, 8u);
                    const Entry e = *reinterpret_cast<const Entry*>(base + (table_at[c] + index * (uint32_t)sizeof(Entry)));
                    if constexpr (LAST) average[c][k] = e;
                    else acc[c][k] += e;
                }
                __builtin_amdgcn_sched_barrier(0);  // (all 16 look-ups in flight would take twice the registers)
            }
        }
    }
    if constexpr (!LAST) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k) average[c][k] = (float)(acc[c][k] * inv_workers);
    }
    float* __restrict__ o = out + (size_t)word0 * 64 + 4u * lane;
    const size_t left = n - (size_t)word0 * 64;  // elements from the span's first one on
    typedef float floatx4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c) {
        const uint32_t e = 256u * c + 4u * lane;
        if (left >= (uint32_t)(kSpanWords * 64) || e + 4u <= left) {  // written once, never re-read here
            const floatx4 x = {average[c][0], average[c][1], average[c][2], average[c][3]};
            __builtin_nontemporal_store(x, reinterpret_cast<floatx4*>(o + 256u * c));
        } else {
#pragma unroll
            for (uint32_t k = 0; k < 4u; ++k)
                if (e + k < left) o[256u * c + k] = average[c][k];
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Bandwidth probes.
// ----------------------------------------------------------------------------------------------
constexpr uint32_t kProbeBlocks = 256 * 8;

__global__ __launch_bounds__(kBlock) void probe_read_kernel(const float4* __restrict__ src, size_t n4,
                                                            float* __restrict__ sink)
{
    float acc = 0.f;
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n4; i += (size_t)gridDim.x * kBlock) {
        const float4 q = src[i];
        acc += (q.x + q.y) + (q.z + q.w);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, kWave);
    if ((threadIdx.x & 63u) == 0) sink[blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6)] = acc;
}

__global__ __launch_bounds__(kBlock) void probe_copy_kernel(const float4* __restrict__ src, float4* __restrict__ dst,
                                                            size_t n4)
{
    for (size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x; i < n4; i += (size_t)gridDim.x * kBlock)
        dst[i] = src[i];
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------
template <int MOST>
static WorkerPtrs<MOST> worker_ptrs(const void* const* d_codes, const float* const* d_levels, uint32_t num_workers)
{
    WorkerPtrs<MOST> ptrs;
    for (uint32_t w = 0; w < (uint32_t)MOST; ++w) {
        ptrs.codes[w] = w < num_workers ? static_cast<const uint64_t*>(d_codes[w]) : nullptr;
        ptrs.levels[w] = w < num_workers ? d_levels[w] : nullptr;
    }
    return ptrs;
}

namespace {

// The arguments of one decode launch; MOST: what its worker list holds.
struct DecodeCall {
    const void* const* codes;
    const float* const* levels;
    uint32_t num_workers;
    size_t n;
    uint32_t words_per_bucket, total_words;
    dim3 grid;
    float* out;
    hipStream_t st;

    template <int MOST, class Kernel>
    void launch(Kernel kernel) const
    {
        launch_kernel(kernel, grid, dim3(kBlock), st, worker_ptrs<MOST>(codes, levels, num_workers), num_workers, n,
                      words_per_bucket, total_words, 1.0 / (double)num_workers, out);
    }
};

// From 512 elements per bucket on only a single worker gets here (launch_by_bucket_size): nothing else is compiled.
template <int BITS, int S, int WPB>
void launch_by_worker(const DecodeCall& call)
{
    if constexpr (WPB < 8) {
        if (call.num_workers > (uint32_t)kFewWorkers) {
            call.launch<OGQ_MAX_WORKERS>(dequantize_average_kernel<BITS, S, WPB, OGQ_MAX_WORKERS>);
            return;
        }
        if (call.num_workers > 1u) {
            call.launch<kFewWorkers>(dequantize_average_kernel<BITS, S, WPB, kFewWorkers>);
            return;
        }
    } else if (call.num_workers > 1u) {
        launch_status() = hipErrorInvalidDeviceFunction;
        return;
    }
    call.launch<1>(dequantize_average_kernel<BITS, S, WPB, 1>);
}

template <int BITS, int S, uint32_t BUCKETS>
void launch_joint_buckets(const DecodeCall& call)
{
    if (call.num_workers <= (BITS > 2 ? 2u : 8u / BITS)) {
        call.launch<kFewWorkers>(dequantize_joint_kernel<BITS, S, BUCKETS, kFewWorkers, true>);
        return;
    }
    if constexpr (BITS > 1) {
        if (call.num_workers <= (uint32_t)kFewWorkers) {
            call.launch<kFewWorkers>(dequantize_joint_kernel<BITS, S, BUCKETS, kFewWorkers, false>);
            return;
        }
    }
    call.launch<OGQ_MAX_WORKERS>(dequantize_joint_kernel<BITS, S, BUCKETS, OGQ_MAX_WORKERS, false>);
}

template <int BITS, int S>
void launch_joint(const DecodeCall& call)
{
    const uint32_t wpb = call.words_per_bucket;
    if (wpb % kSpanWords == 0) launch_joint_buckets<BITS, S, 1>(call);
    else if (wpb > kSpanWords || wpb == 8u) launch_joint_buckets<BITS, S, 2>(call);
    else if (wpb > 8u) launch_joint_buckets<BITS, S, 3>(call);
    else if (wpb > 4u) launch_joint_buckets<BITS, S, 4>(call);
    else launch_joint_buckets<BITS, S, 6>(call);
}

template <int BITS, int S>
void launch_by_bucket_size(const DecodeCall& call)
{
    const uint32_t wpb = call.words_per_bucket;
    const uint32_t fixed = wpb % kSpanWords == 0 ? (uint32_t)kSpanWords : kSpanWords % wpb == 0 ? wpb : 0u;
    // Joint look-ups: bucket sizes that give a span no fixed layout, and several workers from 512 elements on.
    if (fixed == 0u || (wpb >= 8u && call.num_workers > 1u)) {
        launch_joint<BITS, S>(call);
        return;
    }
    switch (fixed) {
        case 16: launch_by_worker<BITS, S, 16>(call); break;
        case 8: launch_by_worker<BITS, S, 8>(call); break;
        case 4: launch_by_worker<BITS, S, 4>(call); break;
        case 2: launch_by_worker<BITS, S, 2>(call); break;
        default: launch_by_worker<BITS, S, 1>(call); break;
    }
}

}  // namespace

void launch_decode(const void* const* d_codes, const float* const* d_levels, uint32_t num_workers, size_t n,
                   const ogq_params_t* p, float* d_out, hipStream_t st)
{
    const uint32_t total_words = (uint32_t)(n / 64 + (n % 64 != 0));
    const uint32_t spans = (total_words + kSpanWords - 1) / kSpanWords;
    const DecodeCall call{d_codes, d_levels, num_workers, n, p->bucket_size / 64, total_words,
                          dim3((spans + kWavesPerBlock - 1) / kWavesPerBlock), d_out, st};
    switch (levels_per_bucket(p->scheme, p->bits)) {
        case 2: launch_by_bucket_size<1, 2>(call); break;
        case 4: launch_by_bucket_size<2, 4>(call); break;
        case 8: launch_by_bucket_size<3, 8>(call); break;
        case 3: launch_by_bucket_size<2, 3>(call); break;
        case 5: launch_by_bucket_size<3, 5>(call); break;
        default: launch_by_bucket_size<4, 9>(call); break;
    }
}

void launch_probe_read(const float* d_src, size_t n, float* d_sink, hipStream_t st)
{
    launch_kernel(probe_read_kernel, dim3(kProbeBlocks), dim3(kBlock), st,
                       reinterpret_cast<const float4*>(d_src), n / 4, d_sink);
}

void launch_probe_copy(const float* d_src, float* d_dst, size_t n, hipStream_t st)
{
    launch_kernel(probe_copy_kernel, dim3(kProbeBlocks), dim3(kBlock), st,
                       reinterpret_cast<const float4*>(d_src), reinterpret_cast<float4*>(d_dst), n / 4);
}

}  // namespace ogq
