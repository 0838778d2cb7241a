// Parameters of the fused layer over neighbour lists (gather_kernel.h, instances in gather_m*.hip).
#pragma once
#include "lists.h"

namespace qgtc {

struct GatherParams {
  // what the sums need, in the order in which it is used
  uint32_t nblocks;
  int32_t run_shift;
  int32_t n_tiles;
  int32_t rows, block;       // rows of the matrix, of a diagonal block (without blocks: all)
  uint32_t block_magic;
  int32_t n_heavy_wg;        // workgroups in front that take the heavy rows
  const int32_t* deg;        // neighbour lists
  const uint16_t* first;
  const uint8_t* X;          // codes as bytes, row-major, minus 128 for eight bits
  int32_t ldx;               // bytes per row (a multiple of 16)
  int32_t cols;              // columns of X
  int32_t self_term;
  int32_t x_offset;          // 128 where X has code - 128
  int32_t h, n_nt, n_ks;     // output columns, 16-column tiles of them, 64-wide steps of K
  int32_t w_off, cols_off, heavy_off;   // LDS: weights (< 0: they do not fit), column sums and terms, what a heavy
                             // row needs; the codes are in front
  int32_t split_y, split_w;  // the operand has 8 bits and is taken as code - 128
  int32_t want_rowsum;
  const uint8_t* wb;         // weights, RIGHT_BYTES
  int64_t wb_part;
  int32_t agg_lo, agg_relu, agg_nbits;   // requantization of the sums
  float agg_inv;
  EpiParams up;
  // rows of more than 16 neighbours; of more than a list holds; heavy rows
  const uint16_t* rest;
  int32_t rest_cap;
  int32_t n_groups;
  const uint64_t* heavy;
  const uint8_t* heavy_cnt;
  const uint32_t* A;
  int64_t lda;
  int32_t a_words;
  int32_t out_flip;          // 0x80808080 where the output is code - 128
  // codes of 9 to 16 bits: the weights' high bytes, bytes they have, parts of the column sums
  const uint8_t* wb_high;
  int32_t w_parts, split_w_high, sum_parts;
};

// What a layer emits.
enum { kGatherCodes = 0, kGatherAffine = 1, kGatherRows = 2,     // codes; behind an affine map; fp32 or int32;
       kGatherSums = 3 };                                        // the sums themselves as fp32 or int32, no second product

// The instances for one kind of output; share: four waves share a tile, else each has one.
// PARTS = 2: codes of 9 to 16 bits.
template <int MODE, int PARTS>
qgtc_status gather_launch(const GatherParams& p, bool share, size_t lds, hipStream_t stream);

// The product of fp32 features, quantized on the way, with weights: first_product.hip.
struct FirstParams {
  GatherParams g;            // rows, cols, weights, epilogue (codes)
  const float* src;
  int64_t ld_src;
  float lo, inv, qmaxf;
};
qgtc_status first_product(FirstParams* p, const qgtc_bits* W, hipStream_t stream);

// What GatherParams says about the weights.
void gather_weights(GatherParams* p, const qgtc_bits* W);

// One layer: p has its operands and epilogues (up.out, up.ld_out: the codes' rows in bytes where
// codes are emitted); W: RIGHT_BYTES.
qgtc_status gather_layer(GatherParams* p, int mode, const qgtc_bits* W, hipStream_t stream);
// The same for codes of 9 to 16 bits, rows of low bytes and behind them high bytes, all minus 128 (ldx is
// twice row_codes_ld()); high: the weights' bits from 8 on, or NULL.
qgtc_status gather_wide_layer(GatherParams* p, int mode, const qgtc_bits* low, const qgtc_bits* high, hipStream_t stream);
qgtc_status pack_wide_rows(const float* src, int64_t ld_src, int rows, int cols, const qgtc_quant* q, uint8_t* dst, hipStream_t stream);
// The aggregation by itself, fp32 or int32 out.
qgtc_status gather_sums(GatherParams* p, hipStream_t stream);

// Rows of codes between the layers of a stack over lists: whole pieces of 16 bytes, code - 128 for
// eight bits (what is past the last column is not used).
inline int64_t row_codes_ld(int cols) { return 16 * (int64_t)cdiv(cols, 16); }
inline uint32_t row_codes_flip(int nbits) { return nbits == 8 ? 0x80808080u : 0u; }

// Features to such rows: Eq. (2) of fp32 (pack.hip), from planes (gather.hip).
qgtc_status pack_row_codes(const float* src, int64_t ld_src, int rows, int cols, const qgtc_quant* q, uint8_t* dst,
                           hipStream_t stream);
// The same and, in the same launch where the features are read 16 bytes at a time, qgtc_pack_weights.
qgtc_status pack_row_codes_and_weights(const qgtc_weight_source* ws, int n, int sums_of, int32_t* col_sums, const float* src, int64_t ld_src,
                                       int rows, int cols, const qgtc_quant* q, uint8_t* dst, hipStream_t stream);
// Checks of features that are quantized into a buffer of a stack.
qgtc_status check_row_codes(const float* src, int rows, int cols, int64_t ld_src, const qgtc_quant* q, const void* buffer, size_t buffer_bytes);
qgtc_status planes_to_rows(const qgtc_bits* X, uint8_t* dst, hipStream_t stream);

}  // namespace qgtc
