// What the two fused layer kernels (layer_kernel.h, gather_kernel.h) share: requantization of the
// aggregated sums to bytes, the weights as operands of the matrix instruction.
#pragma once
#include "agg_mfma.h"

namespace qgtc {
namespace {

// Codes of at most 8 bits: max(c, floor) - lo, with floor = max(lo, 0 with ReLU), is the
// integer part of the rule of QGTC_OUT_BITS for every range.  For lo = 0 negative values have
// code 0 with or without ReLU, which is what the conversion makes of them.
struct Rq {
  int32_t floor, lo;
  float inv, qmaxf;
  bool clip;                                         // fewer than 8 bits: 255 is not the last code
};
__device__ __forceinline__ Rq make_rq(int32_t lo, int relu, float inv, int nbits) {
  return Rq{relu ? max(lo, 0) : lo, lo, inv, (float)((1u << nbits) - 1u), nbits < 8};
}
// Four floats to the four bytes of a word, truncated and saturated: v_cvt_pk_u8_f32 converts,
// saturates and inserts in one instruction, and truncates where the rounding mode says so.
#define QGTC_PK(o, a, b, c, d) \
  "v_cvt_pk_u8_f32 " o ", " a ", 0, 0\n\tv_cvt_pk_u8_f32 " o ", " b ", 1, " o "\n\t" \
  "v_cvt_pk_u8_f32 " o ", " c ", 2, " o "\n\tv_cvt_pk_u8_f32 " o ", " d ", 3, " o "\n\t"
#define QGTC_RTZ "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 3\n\ts_nop 1\n\t"
#define QGTC_RNE "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 0, 2), 0\n\ts_nop 1"
__device__ __forceinline__ void trunc_pack(const float (&f)[1][4], uint32_t (&d)[1]) {
  asm(QGTC_RTZ QGTC_PK("%0", "%1", "%2", "%3", "%4") QGTC_RNE
      : "=&v"(d[0]) : "v"(f[0][0]), "v"(f[0][1]), "v"(f[0][2]), "v"(f[0][3]));
}
__device__ __forceinline__ void trunc_pack(const float (&f)[2][4], uint32_t (&d)[2]) {
  asm(QGTC_RTZ QGTC_PK("%0", "%2", "%3", "%4", "%5") QGTC_PK("%1", "%6", "%7", "%8", "%9") QGTC_RNE
      : "=&v"(d[0]), "=&v"(d[1])
      : "v"(f[0][0]), "v"(f[0][1]), "v"(f[0][2]), "v"(f[0][3]), "v"(f[1][0]), "v"(f[1][1]), "v"(f[1][2]), "v"(f[1][3]));
}
__device__ __forceinline__ void trunc_pack(const float (&f)[4][4], uint32_t (&d)[4]) {
  asm(QGTC_RTZ QGTC_PK("%0", "%4", "%5", "%6", "%7") QGTC_PK("%1", "%8", "%9", "%10", "%11")
      QGTC_PK("%2", "%12", "%13", "%14", "%15") QGTC_PK("%3", "%16", "%17", "%18", "%19") QGTC_RNE
      : "=&v"(d[0]), "=&v"(d[1]), "=&v"(d[2]), "=&v"(d[3])
      : "v"(f[0][0]), "v"(f[0][1]), "v"(f[0][2]), "v"(f[0][3]), "v"(f[1][0]), "v"(f[1][1]), "v"(f[1][2]), "v"(f[1][3]),
        "v"(f[2][0]), "v"(f[2][1]), "v"(f[2][2]), "v"(f[2][3]), "v"(f[3][0]), "v"(f[3][1]), "v"(f[3][2]), "v"(f[3][3]));
}
// The codes of N x 4 sums as N words.
template <int N>
__device__ __forceinline__ void pack_codes_words(const uint32_t (&c)[N][4], const Rq& q, uint32_t (&d)[N]) {
  float f[N][4];
  if (q.lo == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) f[i][r] = (float)(int32_t)c[i][r] * q.inv;
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) f[i][r] = (float)((uint32_t)max((int32_t)c[i][r], q.floor) - (uint32_t)q.lo) * q.inv;
  }
  if (q.clip) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) f[i][r] = fminf(f[i][r], q.qmaxf);
  }
  trunc_pack(f, d);
}

// A block of RIGHT_BYTES (16 output columns, 64 K positions) as the operand of a step of 16 PT K
// positions: lane (ln, g) takes positions 4 PT g .. of output column ln.
template <int PT>
__device__ __forceinline__ v4u load_w(const uint8_t* blk, int lane) {
  v4u v = {0u, 0u, 0u, 0u};
  const int ln = lane & 15, g = lane >> 4;
  if constexpr (PT == 4) {
    v = *reinterpret_cast<const v4u*>(blk + lane * 16);
  } else if constexpr (PT == 2) {
    const v2u a = *reinterpret_cast<const v2u*>(blk + (ln + 16 * (g >> 1)) * 16 + 8 * (g & 1));
    v.x = a.x;
    v.y = a.y;
  } else {
    v.x = *reinterpret_cast<const uint32_t*>(blk + ln * 16 + 4 * g);
  }
  return v;
}

}  // namespace
}  // namespace qgtc
