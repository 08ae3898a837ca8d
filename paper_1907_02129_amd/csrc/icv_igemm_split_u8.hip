// Instantiations of the split-reduction kernel: uint8 x int8.
#include "icv_igemm_split_kernel.h"

namespace icv {

int launch_split_u8(const SplitArgs& a, int tile, int rows, bool tail, hipStream_t s)
{
    return launch_split_instances<ICV_U8I8>(a, tile, rows, tail, s);
}

}  // namespace icv
