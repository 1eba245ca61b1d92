// Vector-unit round kernels, FP32 sampling precision.
#include "hpsmc_round.h"

namespace hpsmc {

hipError_t launch_adv_valu_f32(const RoundArgs &a, int ns, dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    return adv_d<float>(a, ns, grid, block, lds, s);
}

}  // namespace hpsmc
