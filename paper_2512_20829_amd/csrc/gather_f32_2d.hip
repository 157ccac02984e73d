// The gather kernels and launchers for binary32 in 2-D (one unit per precision and
// dimension, so that the instantiations compile in parallel).
#include "gather.hpp"

namespace flp {

template hipError_t launch_gather<float, 2>(const GatherArgs&, int, bool, int, const GatherSpare&, hipStream_t);
template hipError_t launch_gather_batch<float, 2>(const BatchItem*, int, int, int, int, bool, int, bool, uint32_t*, int,
                                             const GatherSpare&, hipStream_t);

}  // namespace flp
