// Two-steps-per-pass kernels of the D3Q27 lattices (central and raw moments).
#include "two_step.hpp"

namespace lbm {

void launch_pair_q27(int precision, bool raw, bool walls, const void* src, void* dst, const Geom& g, const Phys& ph,
                     const PairShape& sh, hipStream_t st)
{
    if (precision == PREC_FP64) {
        if (raw) LaunchPair<LatD3Q27RM, double>::step(walls, false, src, dst, g, ph, sh, 0, st);
        else LaunchPair<LatD3Q27, double>::step(walls, false, src, dst, g, ph, sh, 0, st);
    } else {
        if (raw) LaunchPair<LatD3Q27RM, float>::step(walls, false, src, dst, g, ph, sh, 0, st);
        else LaunchPair<LatD3Q27, float>::step(walls, false, src, dst, g, ph, sh, 0, st);
    }
}

int pair_threads_q27(int precision)
{
    return precision == PREC_FP64 ? pair_threads<LatD3Q27, double>() : pair_threads<LatD3Q27, float>();
}

} // namespace lbm
