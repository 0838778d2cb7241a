// Neighbour lists of a sparse adjacency.
//
// A row's list is blocks of 16 entries (columns of A), the first block of every row side by side, the
// others behind them.  Entry e of a block lies at 4 (e % 4) + e / 4, so that the lane that takes
// entries g, 4 + g, 8 + g, 12 + g reads them as 8 bytes; past the last entry there is kListNone.
// Rows of more than kListLight neighbours ("heavy") are found through a count and a mask per group
// of 64 rows: they are taken by workgroups of their own, or a few hubs would hold up their tiles (the
// subgraph of a power-law graph's hubs can have half of all edges).
#pragma once
#include "agg_mfma.h"

namespace qgtc {

constexpr int kListBlock = 16;
constexpr int kListMax = 256;        // entries that are stored; of more neighbours none is missing in A
constexpr int kListLight = 64;
constexpr int kListNone = 0xffff;    // not a column: those are fewer than 65535
constexpr int kListGroup = 64;       // rows of a group

qgtc_status check_neighbours(const qgtc_neighbours* n, const qgtc_bits* A);

}  // namespace qgtc
