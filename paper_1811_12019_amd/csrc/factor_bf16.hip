// Factor tiles from bf16 tensors (factor_launch.h).
#include "factor_launch.h"

namespace kfac {
template int launch_tiles<0>(int, bool, const FBatch&, hipStream_t);
}  // namespace kfac
