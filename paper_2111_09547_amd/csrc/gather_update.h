// The second product of a layer whose activations are row-major bytes, and its epilogue: codes of a tile of
// 16 rows in LDS ([64 columns][row][64 bytes]) times the weights, weights along M.  Shared by the layers over
// neighbour lists (gather_kernel.h) and by the product of features that comes first (first_product.hip).
#pragma once
#include "gather.h"
#include "layer_parts.h"

namespace qgtc {
namespace {

typedef v4u v4u_a4 __attribute__((aligned(4)));      // 16 bytes at a multiple of four

__device__ __forceinline__ v4i mfma_i8(const v4i& a, const v4i& x, const v4i& c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, x, c, 0, 0, 0); }
// Codes of four columns from col on as they are multiplied: code 0 past the last column, minus 128 for eight bits.
__device__ __forceinline__ uint32_t kept_codes(const GatherParams& p, uint32_t word, int col) {
  return (word & (uint32_t)((1ull << (8 * min(max(p.cols - col, 0), 4))) - 1ull)) ^ (p.split_y ? 0x80808080u : 0u);
}

// Weights as operands (codes, minus 128 for eight bits) into LDS, their sums and the column terms.
template <int LT, int MODE>
__device__ __forceinline__ void stage_weights(const GatherParams& p, uint8_t* lds, int wave, int lane) {
  constexpr bool PERM = LT == 4 && MODE != kGatherRows;
  const int ln = lane & 15, g = lane >> 4;
  const int n_ks = p.n_ks, n_nt = p.n_nt, n_ntp = LT == 4 ? (n_nt + 3) & ~3 : n_nt;
  const bool w8 = p.split_w != 0;
  uint32_t* const wsum = reinterpret_cast<uint32_t*>(lds + p.cols_off);
  double* const colterm = reinterpret_cast<double*>(lds + p.cols_off + n_ntp * 64);
  for (int nt = wave; nt < n_ntp; nt += 4) {
    uint32_t sum = 0u;
    // column c of a group of 64 is position 4 (c / 16) + c % 4 of tile (c / 4) % 4
    const int to = PERM ? ((nt & ~3) + (ln >> 2)) * 1024 + (4 * (nt & 3) + (ln & 3) + 16 * g) * 16 : nt * 1024 + lane * 16;
    for (int ks = 0; ks < n_ks; ++ks) {
      v4u v = {0u, 0u, 0u, 0u};
      if (LT == 1 || nt < n_nt) {
        const uint8_t* blk = p.wb + (int64_t)(nt * n_ks + ks) * 1024;
        v = load_w<4>(blk, lane);
        if (w8) v |= load_w<4>(blk + p.wb_part, lane) << 7;
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) sum = __builtin_amdgcn_sad_u8(v[i], 0u, sum);
      if (w8) v ^= 0x80808080u;
      if (p.w_off >= 0) *reinterpret_cast<v4u*>(lds + p.w_off + ks * n_ntp * 1024 + to) = v;
    }
    sum += (uint32_t)__shfl_xor((int)sum, 16, 64);
    sum += (uint32_t)__shfl_xor((int)sum, 32, 64);
    const int h = nt * 16 + ln;
    if (g == 0) wsum[h] = sum << 7;
    if (MODE == kGatherRows && p.up.mode == QGTC_OUT_F32) {
      const double t = p.up.ck + p.up.cs * (p.up.col_i ? (double)p.up.col_i[min(h, p.h - 1)] : 0.0);
      if (g == 0) colterm[h] = t;
    }
  }
}

// Products of the codes at yb (of the steps ks0 .. ks1 - 1, the first one's in front) with the weights of
// output tiles nt0 .. nt0 + LT - 1 onto z, and their sums onto rs.
template <int LT, int MODE>
__device__ __forceinline__ void add_products(const GatherParams& p, const uint8_t* lds, const uint8_t* yb, int ks0, int ks1, int nt0, bool row_sums,
                                             v4i (&z)[LT], v4i& rs, int lane) {
  constexpr bool PERM = LT == 4 && MODE != kGatherRows;
  const int ln = lane & 15, g = lane >> 4;
  const int n_ntp = LT == 4 ? (p.n_nt + 3) & ~3 : p.n_nt;
  const uint8_t* ya = yb + ln * 64 + g * 16;
  const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
  if (p.w_off >= 0) {
    const uint8_t* w = lds + p.w_off + (ks0 * n_ntp + nt0) * 1024 + lane * 16;
    for (int ks = ks0; ks < ks1; ++ks) {
      const v4i y = *reinterpret_cast<const v4i*>(ya);
      if (row_sums) rs = mfma_i8(ones, y, rs);
#pragma unroll
      for (int j = 0; j < LT; ++j) z[j] = mfma_i8(*reinterpret_cast<const v4i*>(w + j * 1024), y, z[j]);
      ya += 1024;
      w += n_ntp * 1024;
    }
  } else {                                           // too many for LDS
    for (int ks = ks0; ks < ks1; ++ks) {
      const v4i y = *reinterpret_cast<const v4i*>(ya);
      if (row_sums) rs = mfma_i8(ones, y, rs);
#pragma unroll
      for (int j = 0; j < LT; ++j) {
        const int nt = PERM ? nt0 + (ln >> 2) : nt0 + j, l = PERM ? 4 * j + (ln & 3) + 16 * g : lane;
        const uint8_t* blk = p.wb + (int64_t)(min(nt, p.n_nt - 1) * p.n_ks + ks) * 1024;   // (past the last tile: not used)
        v4i wv = *reinterpret_cast<const v4i*>(blk + l * 16);
        if (p.split_w) wv = (wv | *reinterpret_cast<const v4i*>(blk + p.wb_part + l * 16) << 7) ^ (int)0x80808080;
        z[j] = mfma_i8(wv, y, z[j]);
      }
      ya += 1024;
    }
  }
}

// Epilogue of output tiles nt0 .. nt0 + LT - 1 of the 16 rows from row0 on; lane (node n, group g), which
// writes if out_ok.  WHOLE: z and rs are those of the codes, not of the codes minus 128.
template <int LT, int MODE, bool WHOLE = false>
__device__ __forceinline__ void emit_tile(const GatherParams& p, const uint8_t* lds, int row0, bool out_ok, int nt0, v4i (&z)[LT], const v4i& rs,
                                          int32_t rl, int lane) {
  constexpr bool PERM = LT == 4 && MODE != kGatherRows;
  const int ln = lane & 15, g = lane >> 4;
  const int n_nt = p.n_nt, n_ntp = LT == 4 ? (n_nt + 3) & ~3 : n_nt;
  const int out_row = row0 + ln;
  const uint32_t* const wsum = reinterpret_cast<const uint32_t*>(lds + p.cols_off);
  const double* const colterm = reinterpret_cast<const double*>(lds + p.cols_off + n_ntp * 64 * p.sum_parts);
  const EpiParams& u = p.up;
  const Rq oq = make_rq(u.rq_lo, u.relu, u.rq_inv_scale, u.rq_nbits);
  double t1 = 0.0, l0 = 0.0;
  if (MODE == kGatherRows && u.mode == QGTC_OUT_F32) {
    double ri = 0.0;
    if (p.want_rowsum) ri = (double)((uint32_t)rs[0] + (WHOLE || !p.split_y ? 0u : (uint32_t)(p.n_ks * 64) << 7));
    else if (u.row_i && out_ok) ri = (double)u.row_i[out_row];
    t1 = u.rs * ri;
    l0 = u.l0a + u.l0b * (double)rl;
  }
  if (!WHOLE && p.split_w) {
#pragma unroll
    for (int j = 0; j < LT; ++j) z[j] += rs << 7;
  }
  const int h0 = nt0 * 16 + (PERM ? 16 * g : 4 * g);   // first column of the lane, tile 0; the next tile's is HJ further
  constexpr int HJ = PERM ? 4 : 16;
  if (!WHOLE && p.split_y) {
#pragma unroll
    for (int j = 0; j < LT; ++j) z[j] += *reinterpret_cast<const v4i*>(wsum + h0 + HJ * j);
  }
  if constexpr (MODE != kGatherRows) {
    uint32_t d[LT];
    if constexpr (MODE == kGatherAffine) {
      const uint32_t qmax = (uint32_t)oq.qmaxf;
#pragma unroll
      for (int j = 0; j < LT; ++j) {
        d[j] = 0u;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int hc = min(h0 + HJ * j + r, p.h - 1);
          const float ca = u.col_a[hc], cb = u.col_b ? u.col_b[hc] : 0.0f;
          d[j] |= requantize_affine((uint32_t)z[j][r], ca, cb, u.relu, oq.lo, oq.inv, qmax, oq.qmaxf) << (8 * r);
        }
      }
    } else {
      uint32_t c[LT][4];
#pragma unroll
      for (int j = 0; j < LT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) c[j][r] = (uint32_t)z[j][r];
      pack_codes_words(c, oq, d);
    }
    if (out_ok && h0 < (int)u.ld_out) {
      uint8_t* const dst = reinterpret_cast<uint8_t*>(u.out) + (int64_t)out_row * u.ld_out + h0;
      const uint32_t f = (uint32_t)p.out_flip;
      if constexpr (LT == 4) *reinterpret_cast<v4u*>(dst) = (v4u){d[0] ^ f, d[1] ^ f, d[2] ^ f, d[3] ^ f};
      else *reinterpret_cast<uint32_t*>(dst) = d[0] ^ f;
    }
  } else {
#pragma unroll
    for (int j = 0; j < LT; ++j) {
      if (nt0 + j >= n_nt) continue;             // wave-uniform
      const int h = h0 + HJ * j;
      uint32_t res[4];
      if (u.mode == QGTC_OUT_I32) {
#pragma unroll
        for (int r = 0; r < 4; ++r) res[r] = (uint32_t)(u.relu ? max(z[j][r], 0) : z[j][r]);
      } else {
        // the arithmetic of dequantize_f64, with the row and column terms formed once
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double v = (u.cc * (double)z[j][r] + t1) + l0 * colterm[h + r];
          if (u.col_a) {
            const int hc = min(h + r, p.h - 1);
            v = v * (double)u.col_a[hc] + (u.col_b ? (double)u.col_b[hc] : 0.0);
          }
          if (u.relu) v = v < 0.0 ? 0.0 : v;
          res[r] = __float_as_uint((float)v);
        }
      }
      if (out_ok) {
        uint32_t* const dst = reinterpret_cast<uint32_t*>(u.out) + (int64_t)out_row * u.ld_out + h;
        if (h + 4 <= p.h) {
          *reinterpret_cast<v4u_a4*>(dst) = (v4u){res[0], res[1], res[2], res[3]};
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (h + r < p.h) dst[r] = res[r];
        }
      }
    }
  }
}

// Update and epilogue of all output tiles, from nt_first on and every nt_step.
template <int LT, int MODE>
__device__ __forceinline__ void finish_tile(const GatherParams& p, const uint8_t* lds, const uint8_t* yb, int row0, bool out_ok, int nt_first,
                                            int nt_step, int32_t rl, int lane) {
  const v4i zero = {0, 0, 0, 0};
  bool row_sums = p.split_w || (MODE == kGatherRows && p.want_rowsum);
  v4i rs = zero;
#pragma unroll 1
  for (int nt0 = nt_first; nt0 < p.n_nt; nt0 += nt_step) {
    v4i z[LT];
#pragma unroll
    for (int j = 0; j < LT; ++j) z[j] = zero;
    add_products<LT, MODE>(p, lds, yb, 0, p.n_ks, nt0, row_sums, z, rs, lane);
    row_sums = false;                                // (once)
    emit_tile<LT, MODE>(p, lds, row0, out_ok, nt0, z, rs, rl, lane);
  }
}

// ---- codes of 9 to 16 bits: a low and a high byte, both taken as code - 128 -----------------------------
// With y = y0 + 256 y1 and w = w0 + 256 w1 the product is y0 w0 + 256 (y0 w1 + y1 w0) + 65536 y1 w1 modulo 2^32,
// each of them by the instruction for bytes; weights of at most 8 bits have no w1.  Against bit planes (plane
// products with tiles of A, row sums, then s x t one-bit products by popcount, which alone took 25 us of 51): one
// launch of 8 us, and the pass on 8192 rows of 64 columns with 16 bits takes 16 to 20 us in place of 54.

// The codes of the aggregation's results (modulo 2^32) of four columns, as two words of bytes.
__device__ __forceinline__ void wide_bytes(const uint32_t (&c)[4], uint32_t& lo, uint32_t& hi) {
  const uint32_t a = __builtin_amdgcn_perm(c[1], c[0], 0x05010400u), b = __builtin_amdgcn_perm(c[3], c[2], 0x05010400u);   // lo lo hi hi
  lo = __builtin_amdgcn_perm(b, a, 0x05040100u);
  hi = __builtin_amdgcn_perm(b, a, 0x07060302u);
}
__device__ __forceinline__ void wide_codes(const GatherParams& p, const uint32_t (&sum)[4], uint32_t& lo, uint32_t& hi) {
  const uint32_t qmax = (1u << p.agg_nbits) - 1u;
  uint32_t c[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) c[r] = requantize_code(sum[r], p.agg_relu, p.agg_lo, p.agg_inv, qmax, (float)qmax);
  wide_bytes(c, lo, hi);
}

// Byte `part` of the weights of tile nt, step ks: minus 128.
__device__ __forceinline__ v4u wide_weight(const GatherParams& p, int part, int nt, int ks, int lane) {
  const uint8_t* blk = (part == 0 ? p.wb : p.wb_high) + (int64_t)(nt * p.n_ks + ks) * 1024;
  v4u v = load_w<4>(blk, lane);
  if (part == 0 ? p.split_w : p.split_w_high) v |= load_w<4>(blk + p.wb_part, lane) << 7;
  return v;
}
template <int MODE>
__device__ __forceinline__ void stage_wide_weights(const GatherParams& p, uint8_t* lds, int wave, int lane) {
  const int ln = lane & 15, g = lane >> 4;
  const int n_ks = p.n_ks, n_nt = p.n_nt;
  uint32_t* const wsum = reinterpret_cast<uint32_t*>(lds + p.cols_off);   // [part][column]
  double* const colterm = reinterpret_cast<double*>(lds + p.cols_off + n_nt * 128);
  for (int i = wave; i < n_nt * p.w_parts; i += 4) {
    const int nt = i % n_nt, part = i / n_nt;
    uint32_t sum = 0u;
    for (int ks = 0; ks < n_ks; ++ks) {
      v4u v = wide_weight(p, part, nt, ks, lane);
#pragma unroll
      for (int k = 0; k < 4; ++k) sum = __builtin_amdgcn_sad_u8(v[k], 0u, sum);
      if (p.w_off >= 0) *reinterpret_cast<v4u*>(lds + p.w_off + ((part * n_ks + ks) * n_nt + nt) * 1024 + lane * 16) = v ^ 0x80808080u;
    }
    sum += (uint32_t)__shfl_xor((int)sum, 16, 64);
    sum += (uint32_t)__shfl_xor((int)sum, 32, 64);
    const int h = nt * 16 + ln;
    if (g == 0) wsum[part * n_nt * 16 + h] = sum;
    if (MODE == kGatherRows && part == 0 && p.up.mode == QGTC_OUT_F32) {
      const double t = p.up.ck + p.up.cs * (p.up.col_i ? (double)p.up.col_i[min(h, p.h - 1)] : 0.0);
      if (g == 0) colterm[h] = t;
    }
  }
}

template <int MODE>
__device__ __forceinline__ void finish_wide_tile(const GatherParams& p, const uint8_t* lds, const uint8_t* yb, int row0, bool out_ok, int nt_first,
                                                 int nt_step, int32_t rl, int lane) {
  const int ln = lane & 15, g = lane >> 4;
  const int n_ks = p.n_ks, n_nt = p.n_nt;
  const v4i zero = {0, 0, 0, 0}, ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
  const uint8_t* const ya = yb + ln * 64 + g * 16;
  const uint32_t* const wsum = reinterpret_cast<const uint32_t*>(lds + p.cols_off);
  const bool high = p.w_parts == 2;
  v4i r0 = zero, r1 = zero;                          // sums of the codes' bytes, minus 128
  for (int ks = 0; ks < n_ks; ++ks) {
    r0 = mfma_i8(ones, *reinterpret_cast<const v4i*>(ya + ks * 1024), r0);
    r1 = mfma_i8(ones, *reinterpret_cast<const v4i*>(ya + (n_ks + ks) * 1024), r1);
  }
#pragma unroll 1
  for (int nt = nt_first; nt < n_nt; nt += nt_step) {
    v4i z0 = zero, z1 = zero, z2 = zero;
    for (int ks = 0; ks < n_ks; ++ks) {
      const v4i y0 = *reinterpret_cast<const v4i*>(ya + ks * 1024), y1 = *reinterpret_cast<const v4i*>(ya + (n_ks + ks) * 1024);
      v4i w0, w1 = zero;
      if (p.w_off >= 0) {
        w0 = *reinterpret_cast<const v4i*>(lds + p.w_off + (ks * n_nt + nt) * 1024 + lane * 16);
        if (high) w1 = *reinterpret_cast<const v4i*>(lds + p.w_off + ((n_ks + ks) * n_nt + nt) * 1024 + lane * 16);
      } else {                                       // too many for LDS
        w0 = (v4i)(wide_weight(p, 0, nt, ks, lane) ^ 0x80808080u);
        if (high) w1 = (v4i)(wide_weight(p, 1, nt, ks, lane) ^ 0x80808080u);
      }
      z0 = mfma_i8(w0, y0, z0);
      z1 = mfma_i8(w0, y1, z1);
      if (high) {
        z1 = mfma_i8(w1, y0, z1);
        z2 = mfma_i8(w1, y1, z2);
      }
    }
    const int h = nt * 16 + 4 * g;
    const v4i c0 = *reinterpret_cast<const v4i*>(wsum + h);
    // 128 (sum y' + sum w) each, see update_mfma.hip
    z0 += (r0 + c0) << 7;
    z1 += (r1 + c0) << 7;
    if (high) {
      const v4i c1 = *reinterpret_cast<const v4i*>(wsum + n_nt * 16 + h);
      z1 += (r0 + c1) << 7;
      z2 += (r1 + c1) << 7;
    }
    v4i z[1] = {z0 + (z1 << 8) + (z2 << 16)};
    if constexpr (MODE == kGatherRows) {
      const v4i rs = r0 + (r1 << 8) + (int)(257u * 128u * 64u * (uint32_t)n_ks);   // sums of the codes
      emit_tile<1, MODE, true>(p, lds, row0, out_ok, nt, z, rs, rl, lane);
    } else {
      const EpiParams& u = p.up;
      const uint32_t qmax = (1u << u.rq_nbits) - 1u;
      uint32_t c[4], lo, hi;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int hc = min(h + r, p.h - 1);
        if constexpr (MODE == kGatherAffine)
          c[r] = requantize_affine((uint32_t)z[0][r], u.col_a[hc], u.col_b ? u.col_b[hc] : 0.0f, u.relu, u.rq_lo, u.rq_inv_scale, qmax, (float)qmax);
        else
          c[r] = requantize_code((uint32_t)z[0][r], u.relu, u.rq_lo, u.rq_inv_scale, qmax, (float)qmax);
      }
      wide_bytes(c, lo, hi);
      if (out_ok) {
        uint32_t* const dst = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(u.out) + (int64_t)(row0 + ln) * u.ld_out + h);
        dst[0] = lo ^ 0x80808080u;
        dst[u.ld_out / 8] = hi ^ 0x80808080u;
      }
    }
  }
}

}  // namespace
}  // namespace qgtc
