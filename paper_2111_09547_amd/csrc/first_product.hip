// The update in front of the aggregation, A.(X.W), on fp32 features: Eq. (2), the product with the weights and
// the requantization of its result in one pass over the features, which nothing else has to write or read:
// bound by HBM.  262144 x 512 -> 16 (541 MB): 89 us, 6.1 TB/s; quantizer and product as two kernels, with the
// codes written and read in between, 102 and 25 us.
//
// A wave quantizes the 16 rows of a tile, 4 QL columns at a time: QL lanes read 16 bytes each of a row, a
// wave's load is up to 1 KiB in one piece, and all loads of the rows are in flight together.  The codes go
// to LDS as the operand of the matrix instruction (gather_update.h).  Waves walk over tiles, so that the
// weights are put into LDS by few workgroups.
#include "gather_update.h"

namespace qgtc {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef v4f v4f_a4 __attribute__((aligned(4)));

template <int QL, int LT, bool VEC>
__global__ __launch_bounds__(256, 4) void first_product_kernel(const FirstParams fp) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  constexpr int RL = 64 / QL, NL = 16 / RL;          // rows of a load, loads of a tile
  constexpr int CW = 4 * QL, KS = CW / 64;           // columns and steps at a time
  const GatherParams& p = fp.g;
  const int wave = (int)uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int n_ks = p.n_ks;
  stage_weights<LT, kGatherCodes>(p, lds, wave, lane);
  const bool parts = p.n_nt <= LT;                   // one group of output tiles: the codes of CW columns at a time
  uint8_t* const yb = lds + wave * (parts ? KS : n_ks) * 1024;
  const int c4 = 4 * (lane % QL), r_first = lane / QL;
  const bool row_sums = p.split_w != 0;
  __syncthreads();
#pragma unroll 1
  for (int tile = (int)blockIdx.x * 4 + wave; tile < p.n_tiles; tile += (int)gridDim.x * 4) {
    const int row0 = tile * 16;
    v4i z[LT], rs = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < LT; ++j) z[j] = rs;
#pragma unroll 1
    for (int c0 = 0; c0 < p.cols; c0 += CW) {
      const int col = c0 + c4;
      float x[NL][4];
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        // clamped to what exists: no branch around the load
        const float* row = fp.src + (int64_t)min(row0 + i * RL + r_first, p.rows - 1) * fp.ld_src;
        if (VEC) {
          const v4f v = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(row + min(col, p.cols - 4)));
#pragma unroll
          for (int k = 0; k < 4; ++k) x[i][k] = v[k];
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) x[i][k] = row[min(col + k, p.cols - 1)];
        }
      }
      uint32_t d[NL];
#pragma unroll
      for (int i0 = 0; i0 < NL; i0 += 4) {
        float f[4][4];
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int k = 0; k < 4; ++k)                // Eq. (2) with its clamp; a NaN gives 0, truncation is the floor here
            f[i][k] = __builtin_amdgcn_fmed3f((x[i0 + i][k] - fp.lo) * fp.inv, 0.0f, fp.qmaxf);
        trunc_pack(f, w);
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i0 + i] = w[i];
      }
      const int at = parts ? c4 : col;
      if (at < 64 * n_ks) {
#pragma unroll
        for (int i = 0; i < NL; ++i)
          *reinterpret_cast<uint32_t*>(yb + (at >> 6) * 1024 + (i * RL + r_first) * 64 + (at & 63)) = kept_codes(p, d[i], col);
      }
      if (parts) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the lanes read each other's codes
        add_products<LT, kGatherCodes>(p, lds, yb, c0 >> 6, min((c0 >> 6) + KS, n_ks), 0, row_sums, z, rs, lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      }
    }
    const bool out_ok = row0 + (lane & 15) < p.rows;
    if (parts) {
      emit_tile<LT, kGatherCodes>(p, lds, row0, out_ok, 0, z, rs, 0, lane);
    } else {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      finish_tile<LT, kGatherCodes>(p, lds, yb, row0, out_ok, 0, LT, 0, lane);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }
}

template <int QL, int LT>
qgtc_status launch(const FirstParams& p, unsigned grid, size_t lds, hipStream_t stream) {
  const bool vec = p.g.cols % 4 == 0 && p.ld_src % 4 == 0 && ((uintptr_t)p.src & 15u) == 0;
  static OncePerDevice once[2];
  const void* kernel = vec ? reinterpret_cast<const void*>(&first_product_kernel<QL, LT, true>)
                           : reinterpret_cast<const void*>(&first_product_kernel<QL, LT, false>);
  if (!allow_lds(once[vec ? 1 : 0], kernel, lds)) return QGTC_ERR_HIP;
  if (vec) hipLaunchKernelGGL((first_product_kernel<QL, LT, true>), dim3(grid), dim3(256), lds, stream, p);
  else hipLaunchKernelGGL((first_product_kernel<QL, LT, false>), dim3(grid), dim3(256), lds, stream, p);
  return launch_status();
}

}  // namespace

qgtc_status first_product(FirstParams* fp, const qgtc_bits* W, hipStream_t stream) {
  GatherParams& p = fp->g;
  gather_weights(&p, W);
  const int lt = p.n_nt == 1 ? 1 : 4, n_ntp = (p.n_nt + lt - 1) / lt * lt;
  const int ql = p.cols <= 64 ? 16 : (p.cols <= 128 ? 32 : 64);
  size_t lds = (size_t)4 * (p.n_nt <= lt ? ql / 16 : p.n_ks) * 1024;
  p.cols_off = (int)lds;
  lds += (size_t)n_ntp * (64 + 128);
  p.w_off = -1;
  if (p.n_ks * n_ntp <= 48) {
    p.w_off = (int)lds;
    lds += (size_t)p.n_ks * n_ntp * 1024;
  }
  int per_cu = (int)((size_t)(160 * 1024) / (lds + 256));
  if (per_cu > 4) per_cu = 4;
  if (per_cu < 1) per_cu = 1;
  const int64_t wgs = cdiv(p.n_tiles, 4), most = (int64_t)device_compute_units() * per_cu;
  const unsigned grid = (unsigned)(wgs < most ? wgs : most);
  ProfScope prof(QGTC_KERNEL_UPDATE, stream);
  if (ql == 16) return lt == 1 ? launch<16, 1>(*fp, grid, lds, stream) : launch<16, 4>(*fp, grid, lds, stream);
  if (ql == 32) return lt == 1 ? launch<32, 1>(*fp, grid, lds, stream) : launch<32, 4>(*fp, grid, lds, stream);
  return lt == 1 ? launch<64, 1>(*fp, grid, lds, stream) : launch<64, 4>(*fp, grid, lds, stream);
}

}  // namespace qgtc
