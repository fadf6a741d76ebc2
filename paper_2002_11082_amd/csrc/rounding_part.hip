// libogq: one object file per bucket capacity of the random-rounding quantize kernels (the instantiations of
// one capacity take about as long to compile as the rest of the library).  OGQ_PART = 1, 2, 4, 8: one
// wavefront per bucket of at most 256 * OGQ_PART elements (for 2048 elements one wavefront is the faster choice unless
// there are few buckets); 16: four or two wavefronts per bucket of at most 4096 elements; 102: four wavefronts of 2048
// elements per bucket of at most 8192 (22-37 % faster than two wavefronts of 4096: half the registers, twice the resident
// wavefronts); 104, 108: 8, 16 wavefronts of 2048 elements, or 4, 8 of 4096, per bucket of at most 16384, 32768.  ORQ-3 and Linear-3 above
// 4096 elements have a kernel of their own (gather_kernels.h).
#include "rounding_kernels.h"
#include "row_kernels.h"
#include "gather_kernels.h"
#include "pool_kernels.h"

#include "launch.h"

#ifndef OGQ_PART
#error "compile with -DOGQ_PART=<capacity>"
#endif

namespace ogq {

#define OGQ_CAT2(a, b) a##b
#define OGQ_CAT(a, b) OGQ_CAT2(a, b)

// Few buckets: where a gradient has at most a few of them per CU, the time of a call is that of one bucket, and several
// wavefronts per bucket shorten it (64 buckets of 2048, one wavefront and four: eight levels 20.8 -> 14.6 us, three 5.9 ->
// 4.8); beyond, the barriers and the registers of the idle wavefronts cost more than the shorter bucket gains (4096 buckets:
// 38.5 -> 51.1, 14.1 -> 16.8).  profiles/few_buckets_scan.txt has both sides for all rules and sizes.  Each limit up to 2048
// elements, and that above 4096, is a measured number of buckets up to which no rule loses more than 3 % (but BinGrad-pb and three levels 5 and 4 % in
// 1024 of 2048, which the sizes on both sides gain); one number serves all rules, so some would gain further (768 buckets of 1024: BinGrad-pb 6.0 ->
// 6.6, five levels 7.3 -> 6.8).  From 2049 to 4096 elements the other form is two wavefronts, and four lose to it around 2048 buckets, where they begin a
// second round (2048 of 2560: BinGrad-pb 14.6 -> 17.8, the most of any rule that the pool does not take; from 2560 on they gain again, 20.9 -> 20.0).
template <int W, int C>
bool launch_few(uint32_t limit, const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes,
                hipStream_t st)
{
    if (nb > limit) return false;
    launch_orq_team_levels<W, C>(g, n, p, nb, lv, codes, st);
    return true;
}

#if OGQ_PART == 4 || OGQ_PART == 8 || OGQ_PART == 16
// Two or four buckets per workgroup whose levels one wavefront solves side by side (pool_kernels.h), where the solves are what a bucket
// waits for.  What a solve takes in the other kernels depends on the values: their bins suit a mixture of scales and are crowded with Gaussian values, the pool's
// suit both.  The rule takes the pool where it gains on the mean of four kinds of values (mixture, Gaussian, Laplace, Student-t) and of a whole and a
// cut-off last bucket, and not much sooner than it has to: values that few elements share alone (bf16 gradients) send more steps to the general solve, which the
// other kernels do sooner in few buckets (384 of 768, four levels, one sweep, bf16 24 % slower), while half zeros take the pool a third of the time.
// profiles/pool_scan.txt and, with clipping, pool_clip_scan.txt have both sides (crowded values: pool_crowded_scan.txt), and tests/test_dispatch.py holds the rule against them: on the recorded sizes no mean loses
// more than 2 %, no kind of values more than 8 %, and the other kernel is kept nowhere that the mean would gain more than 13 %.  Means, us, other -> pool
// (solves: interior levels, once and for every sweep):
//   eight, nine levels  12 solves and more at every size and number of buckets (18: 64 of 2112 16.5 -> 14.0, 2048 of 1024 24.4 -> 12.6, 12290 of 4096 160 -> 103), fewer up to 1024
//                       elements (16 of 768: 7.7 -> 7.2), to 2048 from 1025 buckets on (768 of 1344: 10.7 -> 11.0, 1026 11.6 -> 11.0), above from 384 (256 of 2112: 10.2 ->
//                       10.9, 384 11.1 -> 10.9), clipped from 1281
//   five levels         12 solves and more likewise (64 of 2112: 13.7 -> 12.3), of 1088 to 1984 elements from 256 on.  Fewer of up to 1024 elements without 4097 to 6144
//                       buckets, where the other kernel still has one round, three from 513 on; clipped 1025 to 4096 buckets.  Of 1088 to 1984 from 1281 on (1026 of 1344:
//                       9.2 -> 9.5, 1282 11.2 -> 9.9) without second_round (clipped, 2816 of 1344: 16.1 -> 16.9).  Above from 1025 (2048), six solves from 384 (of
//                       2112: 11.1 -> 10.5), else from 1281
//   four levels         12 solves and more mostly repeat what they find, which the pool ends early (64 of 4096: 15.8 -> 12.5, 256 of 2048 15.8 -> 12.8).  Up to 1024 elements
//                       from 384 on, four solves from 513, two from 1537 to 5120 buckets (clipped, 4096 of 1024: 11.0 -> 9.5).  Up to 2048 from 1025 on (six solves, whole
//                       2048 from 641, four from 1281), two solves in one round of the pool (4096 of 1344: 15.3 -> 13.1), of whole 2048 from 1281 (clipped, 3072: 15.1 -> 12.9).
//                       Above in full_chip (2 solves of 2112: 16.9 -> 13.2); six solves from 384 or 1025, clipped where three quarters of the registers hold elements (1536 of
//                       4032: 21.6 -> 18.3), four likewise or beyond 3584 (4096 of 3008: 33.2 -> 27.5), two of whole 4096 (8192: 51.6 -> 44.6)
static bool pool_gains(uint32_t d, uint32_t levels, uint64_t solves, uint32_t nb, bool clipped)
{
    const bool second_round = nb > 2560u && nb <= 3072u;  // of the pool up to 2048 elements, where one wavefront per bucket has its first
    const bool full_chip = nb > 1792u && nb <= 2048u;     // above 2048 elements: the pool's first round, the other kernel's second
    const bool fuller = d >= 3584u;
    if (levels >= 8u) return solves >= 12u || d <= 1024u || nb >= (clipped ? 1281u : d > 2048u ? 384u : 1025u);
    if (levels == 5u) {
        if (solves >= 12u) return solves >= 18u || d <= 1024u || d >= 2048u || nb >= 256u;
        if (d <= 1024u) return clipped ? nb > 1024u && nb <= 4096u : (nb <= 4096u || nb > 6144u) && (solves >= 6u || nb > 512u);
        if (d < 2048u) return nb > 1280u && !second_round;
        return nb >= (solves >= 6u && (fuller || (d > 2048u && !clipped)) ? 384u : d == 2048u && !clipped ? 1025u : 1281u);
    }
    if (d > 2048u) {
        if (solves >= 12u) return fuller || nb >= 384u;
        if (full_chip) return true;
        if (solves == 2u) return d == 4096u && nb > 3584u;
        if (solves < 6u) return clipped ? d == 4096u && nb > 1792u : nb > 1280u && (fuller || nb <= 2048u || nb > 3584u);
        return clipped ? fuller && nb > 1280u : nb >= (fuller ? 384u : 1025u);
    }
    if (solves == 2u) return d <= 1024u ? nb > 1536u && nb <= 5120u : d == 2048u ? nb > 1280u : nb > 1792u && nb <= 4096u;
    if (d <= 1024u) return solves >= 12u || nb >= (solves >= 6u ? 384u : 513u);
    if (solves >= 12u) return nb >= (d == 2048u ? 256u : 384u);
    return nb > (solves < 6u ? 1280u : d == 2048u ? 640u : 1024u);
}

template <int W, int C>
static bool launch_pool_part(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if (p->scheme != OGQ_ORQ && p->scheme != OGQ_ORQ_PAPER) return false;
    const uint32_t levels = levels_per_bucket(p->scheme, p->bits);
    const uint64_t solves = (uint64_t)(levels - 2u) * (1u + (uint64_t)p->level_iters);
    if (levels < 4u || !pool_gains(p->bucket_size, levels, solves, nb, p->clip_factor > 0.0f)) return false;
    if (levels == 8u) launch_orq_pool<W, C, 8, 3>(g, n, p, nb, lv, codes, st);
    else if (levels == 9u) launch_orq_pool<W, C, 9, 4>(g, n, p, nb, lv, codes, st);
    else if (levels == 5u) launch_orq_pool<W, C, 5, 3>(g, n, p, nb, lv, codes, st);
    else launch_orq_pool<W, C, 4, 2>(g, n, p, nb, lv, codes, st);
    return true;
}
#endif

#if OGQ_PART == 16
// Four wavefronts of 1024 elements (28 of them in a CU, where two of 2048 make 16) are up to 18 % faster than two on the passes
// over the elements; with BinGrad-pb's long solve that is lost again above some 4000 buckets, which two wavefronts serve better
// (8192 buckets of 4096: 48.9 us with two, 51.4 with four).
void launch_rounding_c16(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if (launch_pool_part<2, 8>(g, n, p, nb, lv, codes, st)) return;
    if (launch_few<4, 4>(p->scheme == OGQ_BINGRAD_PB ? 4096u : ~0u, g, n, p, nb, lv, codes, st)) return;
    launch_orq_team_levels<2, 8>(g, n, p, nb, lv, codes, st);
}
#elif OGQ_PART < 100
#if OGQ_PART <= 2
// Four buckets per wavefront, eight of 128 elements (row_kernels.h), where the gradient has enough of them: a wavefront takes
// longer than one with a single bucket, so where it has a SIMD to itself it only adds latency, unless the solves are what takes long.
// Measured crossover in buckets, on the mean of four kinds of values (profiles/row_kernels_scan.txt; here us, other kernels -> this one):
//   eight and nine levels   of 256 and less elements always (600 buckets of 256, nine levels: 10.4 -> 9.4), above 2048 (2500 of 512,
//                           nine: 13.8 -> 11.4; 2048, where the other kernel's wavefronts just fill the chip: 11.6 -> 11.3), of 128 8192
//   four and five levels    of 256 some 3300 (3500, five: 8.3 -> 6.4), above 4096; four without sweeps, two solves, of 448 and 512 7168 (5120 of
//                           512: 9.4 -> 10.0, 8192: 12.5 -> 11.2), of 128 8192
//   three levels, Linear-s  of 192 3072, of 256 3300 (3072, Linear-3: 4.1 -> 4.2), of 320 and 384 4096, of 448 7168 (5120, Linear-3: 7.0 -> 7.1),
//                           of 512 8192, Linear-3 some 12000 to 16000 (9216: 9.0 -> 9.3), of 128 8192, Linear-5 16384 (12288: 6.3 -> 6.7, 16384: 7.5 -> 7.4)
//                           and Linear-9 65536 (8192: 5.6 -> 7.5, 50000: 19.4 -> 19.8, 65536: 24.3 -> 23.3), as sorted buckets need no search for their
//                           levels; with clipping, which takes the other kernel longer, 12288 (7.3 -> 7.1) and 16384 (9.5 -> 9.4, 12288: 7.9 -> 8.7)
//   no solves               of 320 4096, of 384 and 448 8192 (5120 of 448, nine levels: 5.8 -> 6.7, 8192: 7.7 -> 7.4), of 512 12000 to 16000 (9216:
//                           8.1 -> 9.2), below 8192
static bool launch_row_part(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    const uint32_t levels = levels_per_bucket(p->scheme, p->bits), d = p->bucket_size;
    const bool optimal = (p->scheme == OGQ_ORQ || p->scheme == OGQ_ORQ_PAPER) && levels > 3u;
    const bool even = p->scheme == OGQ_EVEN, solves = !even && levels > 2u;
    const bool two_solves = optimal && levels == 4u && p->level_iters == 0u;
    const uint32_t above_448 = even || (p->scheme == OGQ_LINEAR && levels == 3u) ? 16384u
                               : !optimal ? 8192u
                                          : two_solves ? 7168u : levels < 8u ? 4096u : 2049u;
    const uint32_t above_256 = even && d > 320u ? 8192u
                               : d > 384u && (two_solves || (!optimal && levels < 9u)) ? 7168u
                                                                                      : optimal && levels >= 8u ? 2048u : 4096u;
    const uint32_t above_128 = !solves ? 8192u : optimal && levels >= 8u ? 256u : d > 192u ? 3328u : 3072u;
    const bool clipped = p->clip_factor > 0.0f, more_masses = p->scheme == OGQ_LINEAR && levels > 3u;
    const uint32_t of_128 = !more_masses ? 8192u : levels == 5u ? (clipped ? 12288u : 16384u) : clipped ? 16384u : 65536u;
    const uint32_t enough = d > 448u ? above_448 : d > 256u ? above_256 : d > 128u ? above_128 : of_128;
    if (nb < enough) return false;
#if OGQ_PART == 1
    switch (d) {
        case 64: return false;  // (four buckets per wavefront already: sorted_small_kernel, even_small_kernel)
        case 128:  // eight buckets per wavefront where that leaves two wavefronts per SIMD, with three levels four (four buckets per
                   // wavefront -> eight, us: ORQ-3 9216 buckets 5.3 -> 5.5, 20480 7.3 -> 7.0, 32768 10.1 -> 8.9; ORQ-4 10240 6.9 -> 7.0, 16384 8.6 -> 8.0)
            return nb < (levels > 3u ? 16384u : 32768u) && !more_masses ? launch_rows_levels<16, 2, true>(g, n, p, nb, lv, codes, st) : launch_rows_levels<8, 4, true>(g, n, p, nb, lv, codes, st);
        case 192: return launch_rows_levels<16, 4, false>(g, n, p, nb, lv, codes, st);
        default: return launch_rows_levels<16, 4, true>(g, n, p, nb, lv, codes, st);
    }
#else
    return d == 512 ? launch_rows_levels<16, 8, true>(g, n, p, nb, lv, codes, st)
                    : launch_rows_levels<16, 8, false>(g, n, p, nb, lv, codes, st);
#endif
}
#endif
void OGQ_CAT(launch_rounding_c, OGQ_PART)(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv,
                                          void* codes, hipStream_t st)
{
#if OGQ_PART <= 2
    if (launch_row_part(g, n, p, nb, lv, codes, st)) return;
#endif
#if OGQ_PART == 4 || OGQ_PART == 8
    if (launch_pool_part<1, OGQ_PART>(g, n, p, nb, lv, codes, st)) return;
#endif
#if OGQ_PART == 8
    if (launch_few<4, 2>(1280u, g, n, p, nb, lv, codes, st)) return;
#elif OGQ_PART == 4
    if (launch_few<4, 1>(512u, g, n, p, nb, lv, codes, st)) return;
#elif OGQ_PART == 2
    // one chunk per wavefront: two share the solves of eight or nine levels where the rows above do not take them, nothing else is
    // long enough to share
    if ((p->scheme == OGQ_ORQ || p->scheme == OGQ_ORQ_PAPER) && levels_per_bucket(p->scheme, p->bits) >= 8u &&
        launch_few<2, 1>(~0u, g, n, p, nb, lv, codes, st)) return;
#endif
    launch_orq_levels<OGQ_PART>(g, n, p, nb, lv, codes, st);
}
#elif OGQ_PART == 102
void launch_rounding_w2(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if (launch_few<8, 4>(256u, g, n, p, nb, lv, codes, st)) return;
    if (launch_gather<4, 8>(g, n, p, nb, lv, codes, st)) return;
    launch_orq_team_levels<4, 8>(g, n, p, nb, lv, codes, st);
}
#elif OGQ_PART == 104
void launch_rounding_w4(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if (launch_gather<8, 8>(g, n, p, nb, lv, codes, st)) return;
    // Eight wavefronts of 2048 elements in 128 registers, so that two workgroups put 16 on a CU, where four of 4096 made 8 (1300 buckets of 16384: four
    // levels, two sweeps, 62.8 -> 60.5 us, nine 64.9 -> 62.6, Linear-5 47.2 -> 45.8; 1628 of 12288, Linear-5, 58.0 -> 51.8; but 300 of 16384, five
    // levels, 21.8 -> 22.4).  BinGrad-pb would spill (56.7 -> 80.9).
    if (p->scheme == OGQ_BINGRAD_PB) launch_orq_team<4, 16, 2, 1, kPb>(g, n, p, nb, lv, codes, st);
    else launch_orq_team_levels<8, 8>(g, n, p, nb, lv, codes, st);
}
#elif OGQ_PART == 108
void launch_rounding_w8(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    // Up to one bucket per CU: 16 wavefronts of 2048 elements each; beyond, 8 of 4096, so that two buckets share a CU and one's loads
    // and barriers overlap the other's work (ORQ-3: 512 buckets of 32768 43.6 -> 30.9 us, 782 58.6 -> 44.8, 1562 of 20480 97 -> 75; 256 of
    // 20480 15.2 -> 18.8).
    if (nb <= 256u ? launch_gather<16, 8>(g, n, p, nb, lv, codes, st) : launch_gather<8, 16>(g, n, p, nb, lv, codes, st)) return;
    // Likewise 16 of 2048 where a fifth of 8 of 4096 would hold nothing, and always where the rule has no passes over LDS (8 of 4096 -> 16 of 2048: four
    // levels, two sweeps, 1550 buckets of 16448 132.7 -> 123.3 us, 1000 of 24640 103.6 -> 97.0, clipped 115.8 -> 111.8; Linear-9 107.0 -> 98.1).
    // Above, the gain falls until the buckets fill both (790 of 28672: 106.8 -> 105.8; five levels, clipped, 95.4 -> 97.2).
    if (p->scheme == OGQ_EVEN || (p->scheme != OGQ_BINGRAD_PB && p->bucket_size <= 25600u)) launch_orq_team_levels<16, 8>(g, n, p, nb, lv, codes, st);
    else launch_orq_team_levels<8, 16>(g, n, p, nb, lv, codes, st);
}
#else
#error "unknown OGQ_PART"
#endif

}  // namespace ogq
