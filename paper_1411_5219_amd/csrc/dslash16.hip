// FP16-storage instantiations of the even-odd Dslash kernels.
#include "dslash_impl.h"

namespace lqcd {

hipError_t launch_dslash_16(int recon, int split, bool lnt, bool next, bool dag, int red, const DslashLaunch& L,
                            dim3 grid, dim3 block, hipStream_t s)
{
    if (recon == 12) return launch_hop<16, 12>(split, lnt, next, dag, red, L, grid, block, s);
    return hipErrorInvalidValue;
}

}  // namespace lqcd
