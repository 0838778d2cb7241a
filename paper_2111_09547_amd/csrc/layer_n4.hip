// Fused layer kernel: several column groups of X, up to 64 output columns.
#include "layer_kernel.h"

namespace qgtc {
template qgtc_status layer_launch<4>(const LayerParams&, const AggSplit&, bool, size_t, hipStream_t);
}  // namespace qgtc
