// Instances of the fused layer over neighbour lists for one kind of output.
#include "gather_kernel.h"

namespace qgtc {
template qgtc_status gather_launch<0, 1>(const GatherParams&, bool, size_t, hipStream_t);
}  // namespace qgtc
