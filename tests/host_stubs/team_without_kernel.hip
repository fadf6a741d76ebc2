// Test infrastructure: asks the launchers of the team and one-wavefront kernels for combinations of rule and level count that
// team_serves() and wave_serves() leave uncompiled, and says what status the call ends with.  Nothing is launched and no GPU is needed.
#include <cstdio>

#include "rounding_kernels.h"

namespace ogq {

hipError_t& launch_status()
{
    static thread_local hipError_t status = hipSuccess;
    return status;
}

static int silent = 0, asked = 0;

template <int W, int C, int S, int BITS, int RULE>
void ask()
{
    if constexpr (!team_serves<W, C>(S, RULE)) {
        const ogq_params_t p{};
        launch_status() = hipSuccess;
        launch_orq_team<W, C, S, BITS, RULE>(nullptr, 0, &p, 1u, nullptr, nullptr, nullptr);
        ++asked;
        if (launch_status() == hipSuccess) {
            ++silent;
            printf("no launch and no error: %d wavefronts of %d elements, %d levels, rule %d\n", W, 256 * C, S, RULE);
        }
    }
}

template <int C, int S, int BITS>
void ask_wave()
{
    static_assert(!wave_serves<C>(S, kOptimal), "a combination without a kernel");
    const ogq_params_t p{};
    launch_status() = hipSuccess;
    launch_orq<C, S, BITS, kOptimal>(nullptr, 0, &p, 1u, nullptr, nullptr, nullptr);
    ++asked;
    if (launch_status() == hipSuccess) {
        ++silent;
        printf("no launch and no error: one wavefront of %d elements, %d levels\n", 256 * C, S);
    }
}

template <int W, int C>
void ask_all()
{
    ask<W, C, 2, 1, kPb>();
    ask<W, C, 2, 1, kOptimal>();
    ask<W, C, 4, 2, kOptimal>();
    ask<W, C, 8, 3, kOptimal>();
    ask<W, C, 3, 2, kOptimal>();
    ask<W, C, 5, 3, kOptimal>();
    ask<W, C, 9, 4, kOptimal>();
    ask<W, C, 3, 2, kEven>();
    ask<W, C, 5, 3, kEven>();
    ask<W, C, 9, 4, kEven>();
    ask<W, C, 3, 2, kLinear>();
    ask<W, C, 5, 3, kLinear>();
    ask<W, C, 9, 4, kLinear>();
}

}  // namespace ogq

int main()
{
    using namespace ogq;
    ask_all<2, 1>();
    ask_all<2, 8>();
    ask_all<4, 8>();
    ask_all<4, 16>();
    ask_all<8, 8>();
    ask_all<8, 16>();
    ask_all<16, 8>();
    ask_wave<2, 8, 3>();
    ask_wave<2, 9, 4>();
    ask_wave<4, 8, 3>();
    ask_wave<4, 9, 4>();
    ask_wave<8, 9, 4>();
    printf("%d combinations without a kernel\n", asked);
    return asked == 0 || silent != 0;
}
