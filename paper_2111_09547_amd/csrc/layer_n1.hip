// Fused layer kernel: several column groups of X, up to 16 output columns.
#include "layer_kernel.h"

namespace qgtc {
template qgtc_status layer_launch<1>(const LayerParams&, const AggSplit&, bool, size_t, hipStream_t);
}  // namespace qgtc
