// The gather kernels and launchers for binary64 in 2-D (one unit per precision and
// dimension, so that the instantiations compile in parallel).
#include "gather.hpp"

namespace flp {

template hipError_t launch_gather<double, 2>(const GatherArgs&, int, bool, int, const GatherSpare&, hipStream_t);
template hipError_t launch_gather_batch<double, 2>(const BatchItem*, int, int, int, int, bool, int, bool, uint32_t*, int,
                                             const GatherSpare&, hipStream_t);

}  // namespace flp
