// Parameters of the fused layer kernel and the entry points of its instances.
#pragma once
#include "agg_mfma.h"

namespace qgtc {

struct LayerParams {
  AggParams a;                    // aggregation operands; a.ep: requantization of its result
  EpiParams up;           // epilogue of the update
  const uint8_t* wb;      // weights as bytes in operand order: [part][tile][k step][lane][16]
  int64_t wb_part;        // bytes between the two parts (7 low bits / top bit)
  int32_t h;              // output columns
  int32_t n_nt_w;         // 16-column output tiles
  int32_t n_ks;           // steps along the contraction dimension (64-wide blocks of W)
  int32_t split_y, split_w;   // the operand has 8 bits and is taken as code - 128
  int32_t want_rowsum;
  int32_t w_off, cols_off;    // LDS: weights (< 0: they do not fit), column sums and terms
  int32_t y_off, planes_off;  // LDS: codes of the aggregated rows, packed words of the output
};

// The kernel for one pass over the columns of X (NT = 0), or for several and up to 16 NT output
// columns (NT = 1, 4, 16); one source file each, layer_n*.hip.  codes: X in operand order
// instead of planes.
template <int NT>
qgtc_status layer_launch(const LayerParams& p, const AggSplit& sp, bool codes, size_t lds_bytes, hipStream_t stream);

// The split of a fused layer of `cols` input and `h` output columns over `rows` nodes.
AggSplit layer_split(int rows, int cols, int h, int64_t lda);

// Launch of a layer whose operands (p->a) and epilogues (p->a.ep, p->up) are filled in; W: RIGHT_BYTES.
qgtc_status layer_run(LayerParams* p, const AggSplit& sp, bool codes, const qgtc_bits* W, const qgtc_epilogue* upd_ep, hipStream_t stream);

// ---- activations between the layers of a stack, as codes in operand order ----------------
// Per column group of 16 ct columns and word row (32 nodes): two halves of 16 ct pieces of 16
// bytes.  Piece pos(c) of half h holds the code words 4 h .. 4 h + 3 of column c: code word r
// has the codes of nodes r, r + 8, r + 16, r + 24 of the word row in its bytes 0..3; codes of
// 8-bit operands are stored minus 128.  pos(c) = 16 ((c / 4) % ct) + 4 (c / (4 ct)) + c % 4.
// A stage of the aggregation is a plain copy of this; the layer epilogue writes it directly.
constexpr int kOutCodes = 3;                         // EpiParams.mode; ld_out = log2(ct), ps_out = bytes per column group
__host__ __device__ inline int64_t codes_offset(int c, int ct, int64_t cg_bytes, int64_t word_row) {
  const int cw = 16 * ct, k = c % cw;
  const int pos = 16 * ((k >> 2) % ct) + 4 * (k / (4 * ct)) + (k & 3);
  return (int64_t)(c / cw) * cg_bytes + word_row * (32 * cw) + pos * 16;
}

}  // namespace qgtc
