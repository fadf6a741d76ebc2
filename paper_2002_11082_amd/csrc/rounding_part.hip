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
// wavefronts per bucket shorten it (ORQ-8, one bucket of 2048: 21.4 -> 14.1 us with four; ORQ-3: 5.7 -> 4.2).  Each limit
// is the largest measured number of buckets up to which no rule lost; beyond it the barriers and the registers of the idle
// wavefronts cost more than the shorter bucket gains.
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
// Four wavefronts of 1024 elements (28 of them in a CU, where two of 2048 make 16) are 1 to 12 % faster on the passes over
// the elements; with long serial solves that is lost again above some 4000 buckets, which two wavefronts serve better.
void launch_rounding_c16(const float* g, size_t n, const ogq_params_t* p, uint32_t nb, float* lv, void* codes, hipStream_t st)
{
    if (launch_few<4, 4>(long_solves(p) ? 4096u : ~0u, g, n, p, nb, lv, codes, st)) return;
    launch_orq_team_levels<2, 8>(g, n, p, nb, lv, codes, st);
}
#elif OGQ_PART < 100
#if OGQ_PART <= 2
// Four buckets per wavefront (row_kernels.h) where the gradient has enough of them to fill the chip that way: a
// wavefront then takes about 1.5 times as long as one with a single bucket, so below one wavefront per SIMD (4096
// buckets) it only adds latency.  Measured crossover, in buckets: 2000 to 4000 at 192 and 256 elements, 5000 to 7000 at
// 128 and above 256 (there the LDS holds fewer wavefronts); without level solves about twice that.
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
