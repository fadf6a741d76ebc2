// libogq: one object file per bucket capacity of the random-rounding quantize kernels (the instantiations of
// one capacity take about as long to compile as the rest of the library).  OGQ_PART = 1, 2, 4, 8: one
// wavefront per bucket of at most 256 * OGQ_PART elements (for 2048 elements one wavefront is the faster choice unless
// there are few buckets); 16: four or two wavefronts per bucket of at most 4096 elements; 102: four wavefronts of 2048
// elements per bucket of at most 8192 (22-37 % faster than two wavefronts of 4096: half the registers, twice the resident
// wavefronts); 104, 108: 4, 8 wavefronts of 4096 elements per bucket of at most 16384, 32768.  ORQ-3 and Linear-3 above
// 4096 elements have a kernel of their own, always wavefronts of 2048 elements.
#include "rounding_kernels.h"
#include "row_kernels.h"
#include "gather_kernels.h"

#include "launch.h"

#ifndef OGQ_PART
#error "compile with -DOGQ_PART=<capacity>"
#endif

namespace ogq {

#define OGQ_CAT2(a, b) a##b
#define OGQ_CAT(a, b) OGQ_CAT2(a, b)

// Few buckets: where a gradient has at most a few of them per CU, the time of a call is that of one bucket, and several
// wavefronts per bucket shorten it (64 buckets of 2048, one wavefront and four: eight levels 21.6 -> 14.4 us, three 6.0 ->
// 4.8); beyond, the barriers and the registers of the idle wavefronts cost more than the shorter bucket gains (4096 buckets:
// 39.2 -> 50.0, 13.6 -> 16.2).  profiles/few_buckets_scan.txt has both sides for all rules and sizes.  Each limit is a measured
// number of buckets up to which no rule loses more than 3 %; one number serves all rules, so those with long solves
// would gain somewhat further (1536 buckets of 1024: eight levels 22.8 -> 19.2, where BinGrad-pb loses, 7.4 -> 8.3).
template <int W, int C>
bool launch_few(uint32_t limit, const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes,
                hipStream_t st)
{
    if (nb > limit) return false;
    launch_orq_team_levels<W, C>(g, n, p, nb, lv, codes, st);
    return true;
}

// Rules with many level solves, or BinGrad-pb.
static bool long_solves(const ogq_params_t* p)
{
    return p->scheme == OGQ_BINGRAD_PB ||
           (p->scheme != OGQ_EVEN && p->scheme != OGQ_LINEAR && levels_per_bucket(p->scheme, p->bits) >= 8);
}

#if OGQ_PART == 16
// Four wavefronts of 1024 elements (28 of them in a CU, where two of 2048 make 16) are up to 18 % faster than two on the passes
// over the elements; with long serial solves that is lost again above some 4000 buckets, which two wavefronts serve better
// (8192 buckets of 4096: eight levels 106 us with two, 107 with four, BinGrad-pb 50.8 and 53.4).  The exception that the rule
// leaves alone: around 2048 buckets, one round more for workgroups of four, long solves are faster with two (eight levels
// 31.1 against 37.6).
void launch_rounding_c16(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if (launch_few<4, 4>(long_solves(p) ? 4096u : ~0u, g, n, p, nb, lv, codes, st)) return;
    launch_orq_team_levels<2, 8>(g, n, p, nb, lv, codes, st);
}
#elif OGQ_PART < 100
#if OGQ_PART <= 2
// Four buckets per wavefront (row_kernels.h) where the gradient has enough of them to fill the chip that way: a
// wavefront then takes about 1.5 times as long as one with a single bucket, so below one wavefront per SIMD (4096
// buckets) it only adds latency.  Measured crossover, in buckets (profiles/row_kernels_scan.txt has both sides): 6000 to 8000 at
// 128 elements, against a kernel that already takes two per wavefront; 2000 to 4000 at 192 to 448; up to 8000 at 512, where the
// LDS holds fewer wavefronts.  Without level solves 3000 to 8000, at 128 elements 16000 to 20000.  The limits lie where
// the rules with most solves gain (ORQ-9, 8192 buckets of 512: 23.6 -> 17.1 us; 32768: 73.6 -> 51.9); Linear-5 in buckets of
// 512 loses up to 11 % by them (16384: 17.2 -> 19.1).
static bool launch_row_part(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    const bool solves = p->scheme != OGQ_EVEN && levels_per_bucket(p->scheme, p->bits) > 2;
    const uint32_t d = p->bucket_size;
    const uint32_t enough = d > 256 ? (solves ? 8192u : 16384u) : d > 128 ? (solves ? 4096u : 8192u) : 8192u;
    if (nb < enough) return false;
#if OGQ_PART == 1
    switch (d) {
        case 64: return false;  // (four buckets per wavefront already: sorted_small_kernel, even_small_kernel)
        case 128: return launch_rows_levels<2, true>(g, n, p, nb, lv, codes, st);
        case 192: return launch_rows_levels<4, false>(g, n, p, nb, lv, codes, st);
        default: return launch_rows_levels<4, true>(g, n, p, nb, lv, codes, st);
    }
#else
    return d == 512 ? launch_rows_levels<8, true>(g, n, p, nb, lv, codes, st)
                    : launch_rows_levels<8, false>(g, n, p, nb, lv, codes, st);
#endif
}
#endif
void OGQ_CAT(launch_rounding_c, OGQ_PART)(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv,
                                          void* codes, hipStream_t st)
{
#if OGQ_PART <= 2
    if (launch_row_part(g, n, p, nb, lv, codes, st)) return;
#endif
#if OGQ_PART == 8
    if (launch_few<4, 2>(1280u, g, n, p, nb, lv, codes, st)) return;
#elif OGQ_PART == 4
    if (launch_few<4, 1>(512u, g, n, p, nb, lv, codes, st)) return;
#elif OGQ_PART == 2
    // one chunk per wavefront: two share the solves of eight or nine levels, nothing else is long enough to share
    if (p->scheme != OGQ_BINGRAD_PB && long_solves(p) && launch_few<2, 1>(2560u, g, n, p, nb, lv, codes, st)) return;
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
    if (p->scheme == OGQ_EVEN) {  // no grouping in LDS: half the registers, twice the wavefronts (28 -> 25 us at 25.6 M)
        launch_orq_team_levels<8, 8>(g, n, p, nb, lv, codes, st);
        return;
    }
    launch_orq_team_levels<4, 16>(g, n, p, nb, lv, codes, st);
}
#elif OGQ_PART == 108
void launch_rounding_w8(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if (launch_gather<16, 8>(g, n, p, nb, lv, codes, st)) return;
    if (p->scheme == OGQ_EVEN) {
        launch_orq_team_levels<16, 8>(g, n, p, nb, lv, codes, st);
        return;
    }
    launch_orq_team_levels<8, 16>(g, n, p, nb, lv, codes, st);
}
#else
#error "unknown OGQ_PART"
#endif

}  // namespace ogq
