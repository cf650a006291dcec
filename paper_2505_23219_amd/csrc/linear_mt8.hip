// Instantiations of the skinny linear kernels for up to 128 rows of x.
#include "linear_impl.h"

namespace ghd {

ghd_status launch_linear_mt8(const FusedArgs& a, const LinCut& cut, hipStream_t st)
{
    return launch_linear_r<8, 1>(a, cut, st);
}

}  // namespace ghd
