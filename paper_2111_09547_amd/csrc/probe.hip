// Register-only probe of the AND + popcount rate of the vector ALUs: the inner
// block of the aggregation kernel (v_and_b32 with DPP broadcast + v_bcnt_u32_b32,
// 16 rows x 8 planes) in a loop without any memory traffic.  It gives the
// measured ceiling that the aggregation is priced against beside the nominal one
// (256 CUs x 64 lanes per clock x 2.4 GHz).
// Beside it, on the host: which rows each unit of an aggregation launch takes.
#include "layer.h"

namespace qgtc {
namespace {

#include "popc_blocks.inc"

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void popcount_probe_kernel(int iters, uint32_t* sink) {
  uint32_t acc[16][8];
#pragma unroll
  for (int j = 0; j < 16; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[j][i] = 0u;
  uint32_t x[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = threadIdx.x * 0x9e3779b9u + i;
  uint32_t a = threadIdx.x ^ 0x5bd1e995u;
  for (int k = 0; k < iters; ++k) {
    popc_rows<8>::run(a, x, acc);
    popc_rows<8>::run(a, x, acc);
    popc_rows<8>::run(a, x, acc);
    popc_rows<8>::run(a, x, acc);
  }
  uint32_t v = 0u;
#pragma unroll
  for (int j = 0; j < 16; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) v += acc[j][i];
  if (v == 0x12345678u) sink[0] = v;               // keeps the loop alive; practically never true
}

}  // namespace
}  // namespace qgtc

using namespace qgtc;

extern "C" qgtc_status qgtc_probe_popcount(int32_t workgroups, int32_t waves_per_workgroup, int32_t iters,
                                           uint32_t* sink, void* stream) {
  if (!sink) return QGTC_ERR_NULL;
  if (workgroups < 1 || waves_per_workgroup < 1 || waves_per_workgroup > 4 || iters < 1) return QGTC_ERR_SHAPE;
  hipLaunchKernelGGL(popcount_probe_kernel, dim3((unsigned)workgroups), dim3(64 * waves_per_workgroup), 0,
                     reinterpret_cast<hipStream_t>(stream), iters, sink);
  return launch_status();
}

extern "C" int64_t qgtc_probe_units(const qgtc_bits* A, int32_t x_cols, int32_t out_cols, int64_t first, int64_t count,
                                    int32_t* column, int32_t* row0, int32_t* rows) {
  if (!A || !column || !row0 || !rows || x_cols < 1 || first < 0 || count < 0) return -1;
  qgtc_bits x{};                                     // the shape only
  qgtc_describe(&x, A->block_rows > 0 ? A->rows : A->cols, x_cols, 1, QGTC_RIGHT, 0);
  x.data = A->data;
  AggParams p{};
  if (agg_fill_params(A, nullptr, &x, &p) != QGTC_OK) return -1;
  if (out_cols > 0) {
    (void)agg_set_shape(&p, layer_split(A->rows, x_cols, out_cols, A->ld_words), 1, 0);
  } else {
    const AggSplit sp = aggregate_split(A->rows, x_cols, p.a_words, A->ld_words);
    (void)agg_set_shape(&p, sp, cdiv(x_cols, sp.group()), 0);
  }
  for (int64_t b = first; b < first + count && b < (int64_t)p.nblocks; ++b)
    for (int u = 0; u < kMaxUnits; ++u) {
      AggWave w{};
      w.u = u;
      if (u < p.nu) agg_locate(p, (unsigned)b, &w);
      const int64_t at = (b - first) * kMaxUnits + u;
      column[at] = w.cw;
      row0[at] = w.row0;
      rows[at] = u < p.nu && w.rows_here > 0 ? w.rows_here : 0;
    }
  return p.nblocks;
}
