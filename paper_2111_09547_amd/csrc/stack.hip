// A stack of layers with its activations kept as codes in operand order (layer.h): the
// quantizer writes the first layer's, every hidden layer the next one's, so that staging X
// is a plain copy and no bit plane is formed or put back together between the layers.
#include "gather.h"
#include "layer.h"

#include <cmath>

namespace qgtc {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));

struct CodesParams {
  const float* src;
  int64_t ld_src;
  int32_t rows, cols;
  int32_t ct;                // 16-column tiles per column group
  int64_t cg_bytes;
  uint8_t* dst;
  float lo, inv, qmaxf;
  uint32_t flip;             // 0x80808080 for 8-bit codes
  int32_t n_quads;           // groups of four columns, padding of the last column group included
  uint32_t quad_magic;
};

// Eq. (2) for at most 8 bits: the clamp on the float (a NaN gives 0), truncation of a
// non-negative value is its floor.
__device__ __forceinline__ uint32_t quantize_small(float x, float lo, float inv, float qmaxf) {
  return (uint32_t)__builtin_amdgcn_fmed3f((x - lo) * inv, 0.0f, qmaxf);
}

// Thread (word row kw, half h, four columns): the 16 rows 32 kw + 4 h + {0..3} + 8 {0..3}, four
// columns each, become four code words of four columns: 64 consecutive bytes.  HBM-bound; all
// 16 loads of a thread are in flight together.  VEC: rows are read 16 bytes at a time, and not
// kept in the caches, which then still hold the codes when the first layer reads them (512-16-16
// on 262144 nodes 340 -> 331 us, the five-layer step on 65536 nodes 131 -> 125 us).
template <bool VEC>
__global__ __launch_bounds__(256) void pack_codes_kernel(const CodesParams p) {
  const unsigned idx = blockIdx.x * 256u + threadIdx.x;
  // (the product with the rounded-up reciprocal is at most one too large, for any idx)
  unsigned rest = p.quad_magic ? __umulhi(idx, p.quad_magic) : idx;
  int quad = (int)(idx - rest * (unsigned)p.n_quads);
  if (quad < 0) {
    quad += p.n_quads;
    --rest;
  }
  const int h = (int)(rest & 1u);
  const int kw = (int)(rest >> 1);
  const int r0 = kw * 32 + 4 * h;
  if (kw * 32 >= p.rows) return;
  const int c0 = quad * 4;
  float v[4][4][4];                                  // [byte][word][column]
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* row = p.src + (int64_t)min(r0 + 8 * b + r, p.rows - 1) * p.ld_src;
      if (VEC) {
        const v4f q = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(row + min(c0, p.cols - 4)));
#pragma unroll
        for (int k = 0; k < 4; ++k) v[b][r][k] = q[k];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[b][r][k] = row[min(c0 + k, p.cols - 1)];
      }
    }
  const bool whole = kw * 32 + 32 <= p.rows;
  uint8_t* dst = p.dst + codes_offset(c0, p.ct, p.cg_bytes, kw) + h * 256 * p.ct;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t w[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      w[r] = 0u;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        uint32_t q = quantize_small(v[b][r][k], p.lo, p.inv, p.qmaxf);
        if (!whole && r0 + 8 * b + r >= p.rows) q = 0u;
        w[r] |= q << (8 * b);
      }
      w[r] = (c0 + k < p.cols ? w[r] : 0u) ^ p.flip;
    }
    *reinterpret_cast<uint4*>(dst + 16 * k) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

int64_t codes_cg_bytes(int rows, int ct) { return (int64_t)cdiv(rows, 32) * (512 * ct); }

qgtc_status pack_codes(const float* src, int64_t ld_src, int rows, int cols, const qgtc_quant* q, uint8_t* dst,
                       hipStream_t stream) {
  CodesParams p{};
  p.src = src;
  p.ld_src = ld_src;
  p.rows = rows;
  p.cols = cols;
  p.ct = agg_col_tiles(cols);
  p.cg_bytes = codes_cg_bytes(rows, p.ct);
  p.dst = dst;
  p.lo = (float)q->lo;
  p.inv = qgtc_quant_inv_scale(q->lo, q->hi, q->nbits);
  p.qmaxf = (float)((1u << q->nbits) - 1u);
  p.flip = q->nbits == 8 ? 0x80808080u : 0u;
  p.n_quads = cdiv(cols, 16 * p.ct) * 4 * p.ct;
  p.quad_magic = div_magic(p.n_quads);
  const int64_t items = (int64_t)cdiv(rows, 32) * 2 * p.n_quads;
  const dim3 grid((unsigned)cdiv(items, 256));
  ProfScope prof(QGTC_KERNEL_PACK, stream);
  if (cols % 4 == 0 && ld_src % 4 == 0 && ((uintptr_t)src & 15u) == 0)
    hipLaunchKernelGGL(pack_codes_kernel<true>, grid, dim3(256), 0, stream, p);
  else
    hipLaunchKernelGGL(pack_codes_kernel<false>, grid, dim3(256), 0, stream, p);
  return launch_status();
}

}  // namespace

// One layer of a stack whose operands qgtc_stack_forward has checked: X, or x_codes with x_cols
// columns, in; out_codes, or out, out.
static qgtc_status layer_codes(const qgtc_bits* A, const qgtc_tile_map* map, const qgtc_bits* X, const uint8_t* x_codes,
                        int x_cols, int s, const qgtc_bits* W, const qgtc_epilogue* agg_ep, const qgtc_epilogue* upd_ep,
                        uint8_t* out_codes, void* out, int64_t ld_out, hipStream_t stream) {
  LayerParams p{};
  qgtc_status st;
  if (X) {
    st = agg_fill_params(A, map, X, &p.a);
  } else {
    st = agg_fill_adjacency(A, map, &p.a);
    p.a.X = reinterpret_cast<const uint32_t*>(x_codes);
    p.a.x_bytes = (uint32_t)codes_cg_bytes(A->rows, agg_col_tiles(x_cols));
    p.a.s = s;
    p.a.cols = x_cols;
  }
  if (st != QGTC_OK) return st;
  if (out_codes) {
    EpiParams& u = p.up;
    u.mode = kOutCodes;
    u.relu = upd_ep->relu ? 1 : 0;
    u.rq_nbits = upd_ep->rq_nbits;
    u.rq_lo = upd_ep->rq_lo;
    u.rq_inv_scale = upd_ep->rq_inv_scale;
    u.col_a = upd_ep->col_scale;
    u.col_b = upd_ep->col_shift;
    u.out = out_codes;
    const int ct = agg_col_tiles(W->cols);
    u.ld_out = ct >> 1;                              // (1, 2, 4: 0, 1, 2)
    u.ps_out = codes_cg_bytes(A->rows, ct);
  } else {
    st = make_epilogue(upd_ep, out, ld_out, A->rows, W->cols, QGTC_RIGHT, false, &p.up);
    if (st != QGTC_OK) return st;
  }
  EpiParams& e = p.a.ep;
  e.relu = agg_ep->relu ? 1 : 0;
  e.self_term = agg_ep->self_term ? 1 : 0;
  e.rq_nbits = agg_ep->rq_nbits;
  e.rq_lo = agg_ep->rq_lo;
  e.rq_inv_scale = agg_ep->rq_inv_scale;
  return layer_run(&p, layer_split(A->rows, x_cols, W->cols, A->ld_words), X == nullptr, W, upd_ep, stream);
}

// The operands of an aggregation over neighbour lists: row-major codes of x_cols columns, s bits.
static GatherParams list_operands(const qgtc_bits* A, const qgtc_neighbours* nb, const uint8_t* x_codes, int x_cols, int s) {
  GatherParams p{};
  p.X = x_codes;
  p.first = nb->first;
  p.rest = nb->rest;
  p.deg = nb->deg;
  p.heavy = nb->heavy;
  p.heavy_cnt = nb->heavy_cnt;
  p.n_groups = cdiv(A->rows, kListGroup);
  p.A = A->data;
  p.lda = A->ld_words;
  p.a_words = 4 * cdiv(A->cols, 128);
  p.rest_cap = nb->rest_cap;
  p.rows = A->rows;
  p.block = A->block_rows > 0 ? A->block_rows : A->rows;
  p.block_magic = div_magic(p.block);
  p.n_tiles = cdiv(p.rows, 16);
  p.cols = x_cols;
  p.ldx = (int32_t)row_codes_ld(x_cols);
  p.x_offset = s == 8 ? 128 : 0;
  return p;
}

// Row-major codes as the output of a product of `cols` columns.
static void codes_out(GatherParams* p, const qgtc_epilogue& ep, int cols, uint8_t* out) {
  EpiParams& u = p->up;
  u.mode = QGTC_OUT_BITS;
  u.relu = ep.relu ? 1 : 0;
  u.rq_nbits = ep.rq_nbits;
  u.rq_lo = ep.rq_lo;
  u.rq_inv_scale = ep.rq_inv_scale;
  u.col_a = ep.col_scale;
  u.col_b = ep.col_shift;
  u.out = out;
  u.ld_out = row_codes_ld(cols);
  p->out_flip = (int32_t)row_codes_flip(ep.rq_nbits);
}

// A layer over neighbour lists: row-major codes in; agg: epilogue of the aggregation, upd: of the product
// with W; out_codes, or out, out.
static qgtc_status layer_lists(const qgtc_bits* A, const qgtc_neighbours* nb, const uint8_t* x_codes, int s, const qgtc_epilogue& agg,
                               const qgtc_bits* W, const qgtc_epilogue& upd, uint8_t* out_codes, void* out, int64_t ld_out,
                               hipStream_t stream) {
  GatherParams p = list_operands(A, nb, x_codes, W->rows, s);
  p.self_term = agg.self_term ? 1 : 0;
  p.agg_lo = agg.rq_lo;
  p.agg_relu = agg.relu ? 1 : 0;
  p.agg_nbits = agg.rq_nbits;
  p.agg_inv = agg.rq_inv_scale;
  if (out_codes) {
    codes_out(&p, upd, W->cols, out_codes);
  } else {
    const qgtc_status st = make_epilogue(&upd, out, ld_out, A->rows, W->cols, QGTC_RIGHT, false, &p.up);
    if (st != QGTC_OK) return st;
  }
  return gather_layer(&p, !out_codes ? kGatherRows : (p.up.col_a ? kGatherAffine : kGatherCodes), W, stream);
}

}  // namespace qgtc

using namespace qgtc;

extern "C" size_t qgtc_stack_buffer_bytes(int32_t rows, int32_t cols) {
  if (rows < 0 || cols < 0) return 0;
  const int ct = agg_col_tiles(cols);
  return (size_t)cdiv(cols, 16 * ct) * (size_t)codes_cg_bytes(rows, ct);
}

qgtc_status qgtc::check_row_codes(const float* src, int rows, int cols, int64_t ld_src, const qgtc_quant* q, const void* buffer,
                                  size_t buffer_bytes) {
  if (!src || !q || !buffer) return QGTC_ERR_NULL;
  if (rows < 0 || cols < 0 || ld_src < cols || !(q->hi > q->lo)) return QGTC_ERR_SHAPE;
  if (q->nbits < 1 || q->nbits > 8) return QGTC_ERR_BITWIDTH;
  if (((uintptr_t)buffer & 15u) != 0) return QGTC_ERR_ALIGN;
  if (buffer_bytes < qgtc_stack_buffer_bytes(rows, cols)) return QGTC_ERR_WORKSPACE;
  return QGTC_OK;
}

extern "C" qgtc_status qgtc_stack_input(const float* src, int32_t rows, int32_t cols, int64_t ld_src, const qgtc_quant* q,
                                        void* buffer, size_t buffer_bytes, void* stream) {
  const qgtc_status st = check_row_codes(src, rows, cols, ld_src, q, buffer, buffer_bytes);
  if (st != QGTC_OK || rows == 0 || cols == 0) return st;
  return pack_codes(src, ld_src, rows, cols, q, reinterpret_cast<uint8_t*>(buffer), reinterpret_cast<hipStream_t>(stream));
}

extern "C" qgtc_status qgtc_stack_input_rows(const float* src, int32_t rows, int32_t cols, int64_t ld_src, const qgtc_quant* q,
                                             void* buffer, size_t buffer_bytes, void* stream) {
  const qgtc_status st = check_row_codes(src, rows, cols, ld_src, q, buffer, buffer_bytes);
  if (st != QGTC_OK || rows == 0 || cols == 0) return st;
  return pack_row_codes(src, ld_src, rows, cols, q, reinterpret_cast<uint8_t*>(buffer), reinterpret_cast<hipStream_t>(stream));
}

extern "C" qgtc_status qgtc_stack_input_and_weights(const float* src, int32_t rows, int32_t cols, int64_t ld_src, const qgtc_quant* q,
                                                    void* buffer, size_t buffer_bytes, const qgtc_weight_source* ws, int32_t n,
                                                    int32_t sums_of, int32_t* col_sums, void* stream) {
  const qgtc_status st = check_row_codes(src, rows, cols, ld_src, q, buffer, buffer_bytes);
  if (st != QGTC_OK) return st;
  return pack_row_codes_and_weights(ws, n, sums_of, col_sums, src, ld_src, rows, cols, q, reinterpret_cast<uint8_t*>(buffer),
                                    reinterpret_cast<hipStream_t>(stream));
}

extern "C" qgtc_status qgtc_stack_forward(const qgtc_stack* st, const float* src, int64_t ld_src, const qgtc_quant* q,
                                          const qgtc_bits* X, void* out, int64_t ld_out, void* stream) {
  if (!st || !st->A || !st->layers || !st->buffer[0] || !st->buffer[1]) return QGTC_ERR_NULL;
  if (st->n_layers < 1) return QGTC_ERR_SHAPE;
  if (src) X = nullptr;                              // the features come first
  // Everything is checked before anything is launched, every layer as qgtc_layer checks it.
  AggParams a{};
  qgtc_status rc = agg_fill_adjacency(st->A, st->map, &a);
  if (rc != QGTC_OK) return rc;
  const int rows = st->A->rows;
  if (st->A->block_rows == 0 && st->A->cols != rows) return QGTC_ERR_SHAPE;
  if (agg_long_rows(st->A->ld_words)) return QGTC_ERR_UNSUPPORTED;   // (their split has another order of codes)
  if ((((uintptr_t)st->buffer[0] | (uintptr_t)st->buffer[1]) & 15u) != 0) return QGTC_ERR_ALIGN;
  auto scale_ok = [](float v) { return v > 0.0f && v < INFINITY; };
  for (int l = 0; l < st->n_layers; ++l) {
    const qgtc_stack_layer& y = st->layers[l];
    const bool last = l == st->n_layers - 1;
    rc = check_bits(&y.W, QGTC_RIGHT_BYTES);
    if (rc != QGTC_OK) return rc;
    if (l > 0 && y.W.rows != st->layers[l - 1].W.cols) return QGTC_ERR_SHAPE;
    if (!plan_fused_applies(y.W.rows, y.W.cols, st->s, y.W.nbits)) return QGTC_ERR_UNSUPPORTED;
    if (y.first.mode != QGTC_OUT_BITS || (last ? y.second.mode == QGTC_OUT_BITS : y.second.mode != QGTC_OUT_BITS))
      return QGTC_ERR_UNSUPPORTED;
    if (y.first.col_scale || y.first.col_shift) return QGTC_ERR_UNSUPPORTED;   // the affine map belongs to second
    if (y.second.col_shift && !y.second.col_scale) return QGTC_ERR_NULL;
    if (y.second.self_term) return QGTC_ERR_SHAPE;
    if (y.first.rq_nbits < 1 || y.first.rq_nbits > 8 || (!last && y.second.rq_nbits != st->s)) return QGTC_ERR_BITWIDTH;
    if (!scale_ok(y.first.rq_inv_scale) || (!last && !scale_ok(y.second.rq_inv_scale))) return QGTC_ERR_SHAPE;
    rc = check_tuning(y.second.tuning);
    if (rc != QGTC_OK) return rc;
    // (codes: a column group is addressed with 32 bits)
    if (codes_cg_bytes(rows, agg_col_tiles(y.W.rows)) >= (int64_t)1 << 32) return QGTC_ERR_UNSUPPORTED;
    if (st->buffer_bytes < qgtc_stack_buffer_bytes(rows, y.W.rows)) return QGTC_ERR_WORKSPACE;
  }
  if (!out && rows > 0) return QGTC_ERR_NULL;
  const int d0 = st->layers[0].W.rows;
  if (rows > 0) {
    const qgtc_stack_layer& y = st->layers[st->n_layers - 1];
    EpiParams e{};
    rc = make_epilogue(&y.second, out, ld_out, rows, y.W.cols, QGTC_RIGHT, false, &e);
    if (rc != QGTC_OK) return rc;
  }
  if (X) {
    rc = check_bits(X, QGTC_RIGHT);
    if (rc != QGTC_OK) return rc;
    if (X->rows != rows || X->cols != d0) return QGTC_ERR_SHAPE;
    if (X->nbits != st->s) return QGTC_ERR_BITWIDTH;
    rc = agg_fill_params(st->A, st->map, X, &a);
    if (rc != QGTC_OK) return rc;
  }
  if (st->lists && rows > 0) {
    rc = check_neighbours(st->lists, st->A);
    if (rc != QGTC_OK) return rc;
  }
  if (src) {
    if (q && q->nbits != st->s) return QGTC_ERR_BITWIDTH;
    rc = (st->lists ? qgtc_stack_input_rows : qgtc_stack_input)(src, rows, d0, ld_src, q, st->buffer[0], st->buffer_bytes, stream);
    if (rc != QGTC_OK) return rc;
  }
  if (rows == 0) return QGTC_OK;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  if (st->lists) {
    uint8_t* const codes[2] = {reinterpret_cast<uint8_t*>(st->buffer[0]), reinterpret_cast<uint8_t*>(st->buffer[1])};
    if (X) {
      rc = planes_to_rows(X, codes[0], s);
      if (rc != QGTC_OK) return rc;
    }
    for (int l = 0; l < st->n_layers; ++l) {
      const qgtc_stack_layer& y = st->layers[l];
      rc = layer_lists(st->A, st->lists, codes[l & 1], st->s, y.first, &y.W, y.second, l == st->n_layers - 1 ? nullptr : codes[(l + 1) & 1],
                       out, ld_out, s);
      if (rc != QGTC_OK) return rc;
    }
    return QGTC_OK;
  }
  for (int l = 0; l < st->n_layers; ++l) {
    const qgtc_stack_layer& y = st->layers[l];
    const bool last = l == st->n_layers - 1;
    rc = layer_codes(st->A, st->map, l == 0 ? X : nullptr, reinterpret_cast<const uint8_t*>(st->buffer[l & 1]), y.W.rows,
                     st->s, &y.W, &y.first, &y.second, last ? nullptr : reinterpret_cast<uint8_t*>(st->buffer[(l + 1) & 1]),
                     out, ld_out, s);
    if (rc != QGTC_OK) return rc;
  }
  return QGTC_OK;
}

extern "C" qgtc_status qgtc_stack_forward_update_first(const qgtc_stack* st, const float* src, int64_t ld_src, const qgtc_quant* q,
                                                       void* out, int64_t ld_out, void* stream) {
  if (!st || !st->A || !st->layers || !st->lists || !st->buffer[0] || !st->buffer[1] || !src || !q) return QGTC_ERR_NULL;
  if (st->n_layers < 1) return QGTC_ERR_SHAPE;
  qgtc_status rc = check_adjacency(st->A);
  if (rc != QGTC_OK) return rc;
  const int rows = st->A->rows, d0 = st->layers[0].W.rows;
  if (st->A->block_rows == 0 && st->A->cols != rows) return QGTC_ERR_SHAPE;
  if ((((uintptr_t)st->buffer[0] | (uintptr_t)st->buffer[1]) & 15u) != 0) return QGTC_ERR_ALIGN;
  if (q->nbits != st->s) return QGTC_ERR_BITWIDTH;
  if (ld_src < d0 || !(q->hi > q->lo)) return QGTC_ERR_SHAPE;
  auto scale_ok = [](float v) { return v > 0.0f && v < INFINITY; };
  for (int l = 0; l < st->n_layers; ++l) {
    const qgtc_stack_layer& y = st->layers[l];
    const bool last = l == st->n_layers - 1;
    rc = check_bits(&y.W, QGTC_RIGHT_BYTES);
    if (rc != QGTC_OK) return rc;
    if (l > 0 && y.W.rows != st->layers[l - 1].W.cols) return QGTC_ERR_SHAPE;
    if (!plan_fused_applies(y.W.rows, y.W.cols, st->s, y.W.nbits)) return QGTC_ERR_UNSUPPORTED;
    if (y.first.mode != QGTC_OUT_BITS || (last ? y.second.mode == QGTC_OUT_BITS : y.second.mode != QGTC_OUT_BITS))
      return QGTC_ERR_UNSUPPORTED;
    if (y.first.self_term) return QGTC_ERR_SHAPE;
    if (y.first.col_scale || y.first.col_shift || (!last && (y.second.col_scale || y.second.col_shift))) return QGTC_ERR_UNSUPPORTED;
    if (y.first.rq_nbits != st->s || (!last && y.second.rq_nbits != st->s)) return QGTC_ERR_BITWIDTH;
    if (!scale_ok(y.first.rq_inv_scale) || (!last && !scale_ok(y.second.rq_inv_scale))) return QGTC_ERR_SHAPE;
    rc = check_tuning(y.second.tuning);
    if (rc != QGTC_OK) return rc;
    if (st->buffer_bytes < qgtc_stack_buffer_bytes(rows, y.W.cols)) return QGTC_ERR_WORKSPACE;
  }
  if (rows == 0) return QGTC_OK;
  if (!out) return QGTC_ERR_NULL;
  rc = check_neighbours(st->lists, st->A);
  if (rc != QGTC_OK) return rc;
  const qgtc_stack_layer& end = st->layers[st->n_layers - 1];
  uint8_t* const codes[2] = {reinterpret_cast<uint8_t*>(st->buffer[0]), reinterpret_cast<uint8_t*>(st->buffer[1])};
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  GatherParams sums = list_operands(st->A, st->lists, codes[(st->n_layers - 1) & 1], end.W.cols, st->s);
  sums.self_term = end.second.self_term ? 1 : 0;
  rc = make_epilogue(&end.second, out, ld_out, rows, end.W.cols, QGTC_LEFT, true, &sums.up);
  if (rc != QGTC_OK) return rc;

  FirstParams fp{};
  fp.src = src;
  fp.ld_src = ld_src;
  fp.lo = (float)q->lo;
  fp.inv = qgtc_quant_inv_scale(q->lo, q->hi, q->nbits);
  fp.qmaxf = (float)((1u << q->nbits) - 1u);
  fp.g.rows = rows;
  fp.g.n_tiles = cdiv(rows, 16);
  fp.g.cols = d0;
  fp.g.agg_nbits = st->s;
  codes_out(&fp.g, st->layers[0].first, st->layers[0].W.cols, codes[0]);
  rc = first_product(&fp, &st->layers[0].W, s);
  for (int l = 0; rc == QGTC_OK && l + 1 < st->n_layers; ++l)
    rc = layer_lists(st->A, st->lists, codes[l & 1], st->s, st->layers[l].second, &st->layers[l + 1].W, st->layers[l + 1].first,
                     codes[(l + 1) & 1], nullptr, 0, s);
  return rc == QGTC_OK ? gather_sums(&sums, s) : rc;
}

static size_t wide_bytes_needed(int rows, int cols) { return (size_t)rows * 2 * (size_t)row_codes_ld(cols); }

extern "C" qgtc_status qgtc_wide_input(const float* src, int32_t rows, int32_t cols, int64_t ld_src, const qgtc_quant* q, void* buffer,
                                       size_t buffer_bytes, void* stream) {
  if (!src || !q || !buffer) return QGTC_ERR_NULL;
  if (rows < 0 || cols < 0 || ld_src < cols || !(q->hi > q->lo)) return QGTC_ERR_SHAPE;
  if (rows >= 1 << 24 || cols > 512) return QGTC_ERR_UNSUPPORTED;
  if (q->nbits < 9 || q->nbits > 16) return QGTC_ERR_BITWIDTH;
  if (((uintptr_t)buffer & 15u) != 0) return QGTC_ERR_ALIGN;
  if (buffer_bytes < wide_bytes_needed(rows, cols)) return QGTC_ERR_WORKSPACE;
  if (rows == 0 || cols == 0) return QGTC_OK;
  return pack_wide_rows(src, ld_src, rows, cols, q, reinterpret_cast<uint8_t*>(buffer), reinterpret_cast<hipStream_t>(stream));
}

extern "C" qgtc_status qgtc_wide_forward(const qgtc_wide_stack* st, const float* src, int64_t ld_src, const qgtc_quant* q,
                                         const qgtc_bits* X, void* out, int64_t ld_out, void* stream) {
  if (!st || !st->A || !st->lists || !st->layers || !st->buffer[0] || !st->buffer[1]) return QGTC_ERR_NULL;
  if (st->n_layers < 1) return QGTC_ERR_SHAPE;
  qgtc_status rc = check_adjacency(st->A);
  if (rc != QGTC_OK) return rc;
  const int rows = st->A->rows;
  if (st->A->block_rows == 0 && st->A->cols != rows) return QGTC_ERR_SHAPE;
  if ((((uintptr_t)st->buffer[0] | (uintptr_t)st->buffer[1]) & 15u) != 0) return QGTC_ERR_ALIGN;
  if (st->s < 9 || st->s > 16) return QGTC_ERR_BITWIDTH;
  auto scale_ok = [](float v) { return v > 0.0f && v < INFINITY; };
  for (int l = 0; l < st->n_layers; ++l) {
    const qgtc_wide_layer& y = st->layers[l];
    const bool last = l == st->n_layers - 1, high = y.W[1].data != nullptr;
    for (int i = 0; i < (high ? 2 : 1); ++i) {
      rc = check_bits(&y.W[i], QGTC_RIGHT_BYTES);
      if (rc != QGTC_OK) return rc;
    }
    if (high && (y.W[1].rows != y.W[0].rows || y.W[1].cols != y.W[0].cols)) return QGTC_ERR_SHAPE;
    // (one distance between the two parts of a block for both)
    if (high && y.W[1].nbits == 8 && y.W[1].plane_stride_words != y.W[0].plane_stride_words) return QGTC_ERR_SHAPE;
    if (high && y.W[0].nbits != 8) return QGTC_ERR_BITWIDTH;
    if (l > 0 && y.W[0].rows != st->layers[l - 1].W[0].cols) return QGTC_ERR_SHAPE;
    if (y.W[0].rows < 1 || y.W[0].rows > 512 || y.W[0].cols < 1 || y.W[0].cols > 256) return QGTC_ERR_UNSUPPORTED;
    if (y.first.mode != QGTC_OUT_BITS || (last ? y.second.mode == QGTC_OUT_BITS : y.second.mode != QGTC_OUT_BITS)) return QGTC_ERR_UNSUPPORTED;
    if (y.first.col_scale || y.first.col_shift) return QGTC_ERR_UNSUPPORTED;   // the affine map belongs to second
    if (y.second.col_shift && !y.second.col_scale) return QGTC_ERR_NULL;
    if (y.second.self_term) return QGTC_ERR_SHAPE;
    if (y.first.rq_nbits < 9 || y.first.rq_nbits > 16 || (!last && y.second.rq_nbits != st->s)) return QGTC_ERR_BITWIDTH;
    if (!scale_ok(y.first.rq_inv_scale) || (!last && !scale_ok(y.second.rq_inv_scale))) return QGTC_ERR_SHAPE;
    rc = check_tuning(y.second.tuning);
    if (rc != QGTC_OK) return rc;
    if (st->buffer_bytes < wide_bytes_needed(rows, y.W[0].rows)) return QGTC_ERR_WORKSPACE;
  }
  if (rows >= 1 << 24 || st->A->ld_words >= 1 << 24) return QGTC_ERR_UNSUPPORTED;
  if (src && q && q->nbits != st->s) return QGTC_ERR_BITWIDTH;
  if (src) X = nullptr;                              // the features come first
  if (X) {
    rc = check_bits(X, QGTC_RIGHT);
    if (rc != QGTC_OK) return rc;
    if (X->rows != rows || X->cols != st->layers[0].W[0].rows) return QGTC_ERR_SHAPE;
    if (X->nbits != st->s) return QGTC_ERR_BITWIDTH;
  }
  if (rows == 0) return QGTC_OK;
  if (!out) return QGTC_ERR_NULL;
  rc = check_neighbours(st->lists, st->A);
  if (rc != QGTC_OK) return rc;
  const qgtc_wide_layer& end = st->layers[st->n_layers - 1];
  EpiParams last_ep{};
  rc = make_epilogue(&end.second, out, ld_out, rows, end.W[0].cols, QGTC_RIGHT, false, &last_ep);
  if (rc != QGTC_OK) return rc;
  if (src) {
    rc = qgtc_wide_input(src, rows, st->layers[0].W[0].rows, ld_src, q, st->buffer[0], st->buffer_bytes, stream);
    if (rc != QGTC_OK) return rc;
  }
  if (X) {
    rc = planes_to_rows(X, reinterpret_cast<uint8_t*>(st->buffer[0]), reinterpret_cast<hipStream_t>(stream));
    if (rc != QGTC_OK) return rc;
  }
  uint8_t* const codes[2] = {reinterpret_cast<uint8_t*>(st->buffer[0]), reinterpret_cast<uint8_t*>(st->buffer[1])};
  for (int l = 0; l < st->n_layers; ++l) {
    const qgtc_wide_layer& y = st->layers[l];
    const bool last = l == st->n_layers - 1;
    GatherParams p = list_operands(st->A, st->lists, codes[l & 1], y.W[0].rows, 8);
    p.ldx *= 2;
    p.self_term = y.first.self_term ? 1 : 0;
    p.agg_lo = y.first.rq_lo;
    p.agg_relu = y.first.relu ? 1 : 0;
    p.agg_nbits = y.first.rq_nbits;
    p.agg_inv = y.first.rq_inv_scale;
    if (last) {
      p.up = last_ep;
    } else {
      codes_out(&p, y.second, y.W[0].cols, codes[(l + 1) & 1]);
      p.up.ld_out *= 2;
    }
    rc = gather_wide_layer(&p, last ? kGatherRows : (p.up.col_a ? kGatherAffine : kGatherCodes), &y.W[0], y.W[1].data ? &y.W[1] : nullptr,
                           reinterpret_cast<hipStream_t>(stream));
    if (rc != QGTC_OK) return rc;
  }
  return QGTC_OK;
}
