// Instantiations of the split-reduction kernel: bfloat16.
#include "icv_igemm_split_kernel.h"

namespace icv {

int launch_split_bf16(const SplitArgs& a, int tile, int rows, bool tail, hipStream_t s)
{
    return launch_split_instances<ICV_BF16>(a, tile, rows, tail, s);
}

}  // namespace icv
