// FP64-storage instantiations of the Dslash kernels on several right-hand sides.
#include "hop_rhs.h"

namespace lqcd {

hipError_t launch_rhs_64(int recon, int halves, bool dag, int red, const DslashLaunch& L, dim3 grid, dim3 block, hipStream_t s)
{
    if (recon == 18) return launch_rhs<64, 18>(halves, dag, red, L, grid, block, s);
    if (recon == 12) return launch_rhs<64, 12>(halves, dag, red, L, grid, block, s);
    return hipErrorInvalidValue;
}

}  // namespace lqcd
