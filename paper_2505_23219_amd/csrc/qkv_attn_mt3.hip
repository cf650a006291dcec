// Instantiations of the QKV + attention kernel for up to 48 rows of x.
#include "qkv_attn_impl.h"

namespace ghd {

ghd_status launch_qkv_attn_mt3(const FusedArgs& a, const LinCut& cut, hipStream_t st)
{
    return launch_qkv_attn_r<3, 3>(a, cut, st);
}

}  // namespace ghd
