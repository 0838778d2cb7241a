// Aggregation of long rows on the 4- and 6-bit floating-point matrix instructions: agg_dense.hip.
#pragma once
#include "agg_mfma.h"

namespace qgtc {

// Whether every sum of it is exact there, and the room for X as its operands.
bool dense_applies(const AggParams& p);
int64_t dense_bytes(const AggParams& p);
// Workgroups of so many rows.
int64_t dense_groups(const AggParams& p, int rows);
// p: operands, map and epilogue.
qgtc_status dense_aggregate(const AggParams& p, void* workspace, int xcd_run, hipStream_t stream);

}  // namespace qgtc
