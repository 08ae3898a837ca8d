// Instantiations of the any-channel-count kernel: uint8 x int8.
#include "icv_igemm_any_kernel.h"

namespace icv {

int launch_any_u8(const AnyArgs& a, int variant, int tail, bool fused, hipStream_t s)
{
    return launch_any_instances<ICV_U8I8>(a, variant, tail, fused, s);
}

}  // namespace icv
