// Fused layer kernel, one column group of X.
#include "layer_kernel.h"

namespace qgtc {
template qgtc_status layer_launch<0>(const LayerParams&, const AggSplit&, bool, size_t, hipStream_t);
}  // namespace qgtc
