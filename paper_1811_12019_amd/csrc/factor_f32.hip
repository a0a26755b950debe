// Factor tiles from fp32 tensors (factor_launch.h).
#include "factor_launch.h"

namespace kfac {
template int launch_tiles<2>(int, bool, const FBatch&, hipStream_t);
}  // namespace kfac
