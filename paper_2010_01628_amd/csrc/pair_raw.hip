// Two-steps-per-pass kernels of the D3Q19 raw-moment variant (N = I).
#include "two_step.hpp"

namespace lbm {

void launch_pair_q19rm(int precision, bool walls, bool general, const void* src, void* dst, const Geom& g,
                       const Phys& ph, const PairShape& sh, uint32_t key2, hipStream_t st)
{
    switch (precision) {
    case PREC_FP64: LaunchPair<LatD3Q19RM, double>::step(walls, general, src, dst, g, ph, sh, key2, st); break;
    case PREC_FP32: LaunchPair<LatD3Q19RM, float>::step(walls, general, src, dst, g, ph, sh, key2, st); break;
    case PREC_FP16: LaunchPair<LatD3Q19RM, _Float16>::step(walls, general, src, dst, g, ph, sh, key2, st); break;
    default: LaunchPair<LatD3Q19RM, bf16_t>::step(walls, general, src, dst, g, ph, sh, key2, st); break;
    }
}

} // namespace lbm
