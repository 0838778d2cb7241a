// Instances of the fused layer over neighbour lists for codes of 9 to 16 bits.
#include "gather_kernel.h"

namespace qgtc {
template qgtc_status gather_launch<kGatherCodes, 2>(const GatherParams&, bool, size_t, hipStream_t);
template qgtc_status gather_launch<kGatherAffine, 2>(const GatherParams&, bool, size_t, hipStream_t);
template qgtc_status gather_launch<kGatherRows, 2>(const GatherParams&, bool, size_t, hipStream_t);
}  // namespace qgtc
