// Host side of the fused layer (layer_kernel.h): checks, weights in operand order, launch
// shape and dispatch.
#include "layer.h"

#include <cmath>

namespace qgtc {
namespace {

// Weights: packed planes -> bytes in the operand order of the matrix instruction.
// Thread (tile nt, step ks, lane l) writes the 16 bytes of column 16 nt + l % 16,
// K positions 64 ks + 16 (l / 16) .. + 15.
__global__ __launch_bounds__(256) void weight_bytes_kernel(const uint32_t* W, int64_t ldw, int64_t psw,
                                                           int t, int kwords, int cols, int n_nt_w,
                                                           int n_ks, int split_w, uint8_t* wb,
                                                           int64_t wb_part) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int lane = idx & 63;
  const int ks = (idx >> 6) % n_ks;
  const int nt = (idx >> 6) / n_ks;
  if (nt >= n_nt_w) return;
  const int col = nt * 16 + (lane & 15);
  const int k0 = ks * 64 + (lane >> 4) * 16;
  const int kw = k0 >> 5;
  const int sh = k0 & 31;
  uint32_t f[8];
#pragma unroll
  for (int pl = 0; pl < 8; ++pl) {
    f[pl] = 0u;
    if (pl < t && col < cols && kw < kwords)
      f[pl] = (W[(int64_t)pl * psw + (int64_t)kw * ldw + col] >> sh) & 0xffffu;
  }
  uint32_t d[4];
  planes_to_bytes(f, t, d);
  v4u lo = {d[0], d[1], d[2], d[3]};
  uint8_t* dst = wb + (int64_t)idx * 16;
  if (split_w) {
    v4u hi = (lo >> 7) & 0x01010101u;
    lo = lo & 0x7f7f7f7fu;
    *reinterpret_cast<v4u*>(dst + wb_part) = hi;
  }
  *reinterpret_cast<v4u*>(dst) = lo;
}

}  // namespace

size_t layer_fused_workspace_bytes(int32_t in_cols, int32_t out_cols) {
  // two parts of ceil(out/16) x ceil(in/64) operand blocks of 1 KiB
  return (size_t)2 * (size_t)cdiv(out_cols, 16) * (size_t)cdiv(in_cols, 64) * 1024;
}

qgtc_status layer_fused(const qgtc_bits* A, const qgtc_tile_map* map, const qgtc_bits* X,
                        const qgtc_bits* W, const qgtc_epilogue* agg_ep, const qgtc_epilogue* upd_ep,
                        void* workspace, size_t workspace_bytes, void* out, int64_t ld_out,
                        hipStream_t stream, bool* done) {
  *done = false;
  if (!A || !X || !W || !agg_ep || !upd_ep || !workspace || !out) return QGTC_OK;
  const qgtc_tuning* tn = upd_ep->tuning;
  if (tn && tn->layer_path == 1 && W->layout != QGTC_RIGHT_BYTES) return QGTC_OK;
  // what the kernel covers; everything else takes the two-kernel path
  if (!plan_fused_applies(X->cols, W->cols, X->nbits, W->nbits)) return QGTC_OK;
  if (agg_ep->rq_nbits < 1 || agg_ep->rq_nbits > 8) return QGTC_OK;
  if (upd_ep->mode == QGTC_OUT_BITS && upd_ep->rq_nbits > 8) return QGTC_OK;
  if (A->rows < 1) return QGTC_OK;
  const bool w_bytes = W->layout == QGTC_RIGHT_BYTES;
  if (!w_bytes && workspace_bytes < layer_fused_workspace_bytes(X->cols, W->cols)) return QGTC_OK;
  if (!(agg_ep->rq_inv_scale > 0.0f) || !(agg_ep->rq_inv_scale < INFINITY)) return QGTC_OK;

  LayerParams p{};
  if (agg_fill_params(A, map, X, &p.a) != QGTC_OK) return QGTC_OK;
  if (check_bits(W, w_bytes ? QGTC_RIGHT_BYTES : QGTC_RIGHT) != QGTC_OK || W->rows != X->cols) return QGTC_OK;
  const bool square = A->block_rows > 0 || A->rows == A->cols;
  if (agg_ep->self_term && !square) return QGTC_OK;
  if (make_epilogue(upd_ep, out, ld_out, A->rows, W->cols, QGTC_RIGHT, false, &p.up) != QGTC_OK)
    return QGTC_OK;

  EpiParams& ea = p.a.ep;
  ea = EpiParams{};
  ea.mode = QGTC_OUT_BITS;
  ea.relu = agg_ep->relu ? 1 : 0;
  ea.self_term = agg_ep->self_term ? 1 : 0;
  ea.rq_nbits = agg_ep->rq_nbits;
  ea.rq_lo = agg_ep->rq_lo;
  ea.rq_inv_scale = agg_ep->rq_inv_scale;

  const AggSplit sp = layer_split(A->rows, X->cols, W->cols, A->ld_words);
  if (w_bytes) {
    *done = true;
    return layer_run(&p, sp, false, W, upd_ep, stream);
  }
  // planes: into operand order first
  const int n_nt = cdiv(W->cols, 16), n_ks = cdiv(W->rows, 64);
  qgtc_bits wb = *W;
  wb.data = reinterpret_cast<uint32_t*>(workspace);
  wb.layout = QGTC_RIGHT_BYTES;
  wb.ld_words = 256 * (int64_t)n_ks;
  wb.plane_stride_words = (int64_t)n_nt * wb.ld_words;
  {
    ProfScope prof(QGTC_KERNEL_SUMS, stream);
    hipLaunchKernelGGL(weight_bytes_kernel, dim3((unsigned)cdiv(n_nt * n_ks * 64, 256)), dim3(256), 0, stream, W->data,
                       W->ld_words, W->plane_stride_words, W->nbits, cdiv(W->rows, 32), W->cols, n_nt, n_ks,
                       W->nbits == 8 ? 1 : 0, reinterpret_cast<uint8_t*>(workspace), wb.plane_stride_words * 4);
    qgtc_status st = launch_status();
    if (st != QGTC_OK) return st;
  }
  *done = true;
  return layer_run(&p, sp, false, &wb, upd_ep, stream);
}

// Two waves per unit where 256 rows per workgroup still give every compute unit one, four below
// (and for more than 64 output columns behind several passes, whose accumulators do not fit
// otherwise); the columns are split as evenly as 16-column tiles allow.
AggSplit layer_split(int rows, int cols, int h, int64_t lda) {
  const bool many = (int64_t)cdiv(rows, kUnitRows) >= (int64_t)kMaxUnits * device_compute_units();
  if (cols <= 16 && !agg_long_rows(lda)) return AggSplit{1, 1, 1, 1};
  if (cols <= 32) return AggSplit{1, 2, 2, 1};
  if (cols <= 64) return many ? AggSplit{2, 2, 4, 1} : AggSplit{1, 4, 4, 1};
  return many && (cols <= 128 || h <= 64) ? AggSplit{4, 2, 4, 1} : AggSplit{2, 4, 4, 1};
}

// Launch of a layer whose operands and epilogues are filled in.
qgtc_status layer_run(LayerParams* lp, const AggSplit& sp, bool codes, const qgtc_bits* W, const qgtc_epilogue* upd_ep,
                      hipStream_t stream) {
  LayerParams& p = *lp;
  const qgtc_tuning* tn = upd_ep->tuning;
  size_t lds = agg_set_shape(&p.a, sp, 1, tn ? tn->agg_xcd_run : 0);
  // The aggregated codes, and behind them the packed words of the output, take the place of the
  // stages where one pass is all; with several passes the next one's stages are on their way by then.
  const bool one = p.a.n_pass == 1;
  const size_t y = (size_t)p.a.nu * kUnitRows * sp.group();
  const size_t planes = p.up.mode == QGTC_OUT_BITS ? (size_t)p.a.nu * 2 * 8 * W->cols * 4 : 0;
  if (one) {
    p.y_off = 0;
    p.planes_off = (int)y;
    if (lds < y + planes) lds = y + planes;
  } else {
    lds = (lds + 15) & ~(size_t)15;
    p.y_off = (int)lds;
    lds += y;
    p.planes_off = 0;
    if (lds < planes) lds = planes;
  }
  p.wb = reinterpret_cast<const uint8_t*>(W->data);
  p.wb_part = W->plane_stride_words * 4;
  p.h = W->cols;
  p.n_nt_w = cdiv(W->cols, 16);
  p.n_ks = cdiv(W->rows, 64);
  // weights in operand order (up to 32 KiB), their column sums, fp64 column terms
  lds = (lds + 15) & ~(size_t)15;
  p.cols_off = (int)lds;
  lds += (size_t)p.n_nt_w * (64 + 128);
  p.w_off = -1;
  if (p.n_ks * p.n_nt_w <= 32 && lds + (size_t)p.n_ks * p.n_nt_w * 1024 <= 160 * 1024) {
    p.w_off = (int)lds;
    lds += (size_t)p.n_ks * p.n_nt_w * 1024;
  }
  if (p.up.l0b == 0.0) p.up.row_l = nullptr;
  p.want_rowsum = p.up.mode == QGTC_OUT_F32 && p.up.row_i == nullptr && p.up.rs != 0.0;
  p.split_y = p.a.ep.rq_nbits == 8;
  p.split_w = W->nbits == 8;
  ProfScope prof(QGTC_KERNEL_LAYER, stream);
  if (one) return layer_launch<0>(p, sp, codes, lds, stream);
  if (p.n_nt_w <= 1) return layer_launch<1>(p, sp, codes, lds, stream);
  if (p.n_nt_w <= 4) return layer_launch<4>(p, sp, codes, lds, stream);
  return layer_launch<16>(p, sp, codes, lds, stream);
}

}  // namespace qgtc
