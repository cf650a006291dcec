// Instantiations of the skinny linear kernels for up to 48 rows of x.
#include "linear_impl.h"

namespace ghd {

ghd_status launch_linear_mt3(const FusedArgs& a, const LinCut& cut, hipStream_t st)
{
    return launch_linear_r<3, 1>(a, cut, st);
}

}  // namespace ghd
