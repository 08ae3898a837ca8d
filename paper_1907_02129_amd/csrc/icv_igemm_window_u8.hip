// uint8 instantiations of the window kernel.
#include "icv_igemm_window_kernel.h"

namespace icv {

int launch_window_u8(const WindowArgs& a, int tile, int unroll, size_t lds_bytes, bool fused, hipStream_t s)
{
    return launch_window_instances<ICV_U8I8>(a, tile, unroll, lds_bytes, fused, s);
}

}  // namespace icv
