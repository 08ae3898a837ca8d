// Instantiations of the any-channel-count kernel: fp32.
#include "icv_igemm_any_kernel.h"

namespace icv {

int launch_any_f32(const AnyArgs& a, int variant, int tail, bool fused, hipStream_t s)
{
    return launch_any_instances<ICV_F32>(a, variant, tail, fused, s);
}

}  // namespace icv
