// Factor tiles from fp16 tensors (factor_launch.h).
#include "factor_launch.h"

namespace kfac {
template int launch_tiles<1>(int, bool, const FBatch&, hipStream_t);
}  // namespace kfac
