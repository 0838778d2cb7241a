// One quantized GNN layer in a single kernel (Algorithm 1 of the paper with the
// inter-layer fusion of Section 4.5 taken one step further): neighbour aggregation,
// requantization, node update and the output epilogue, all products on the int8 matrix
// cores, the aggregated tile never leaving the registers.
//
//   1. Aggregation of G = 16 CT WAYS columns (agg_mfma.h): lane (n, g) of a wave ends up with
//      4 CT consecutive columns of node n of each of the unit's four 16-row tiles.
//   2. Requantization to codes of at most 8 bits, four consecutive columns per register.  The
//      waves of a unit put them together in LDS, in the operand order of the matrix
//      instruction: [64 columns][64 rows][64 bytes].
//   3. Update: v_mfma_i32_16x16x64_i8 of the codes (nodes along M; each wave takes 4 / WAYS
//      tiles of the unit) and the weights as bytes (RIGHT_BYTES, kept in LDS).  Operands of
//      8 bits are taken as code - 128, and
//        sum y w = sum y' w' + 128 (sum y' + sum w)    (both), with sum y' from one more
//      instruction against an all-ones operand and sum w taken while W is loaded.
//   4. Epilogue.  ROWS (int32, dequantized fp32): the weights are the operand along M, so that a lane
//      has four consecutive columns of one node and stores 16 bytes (with single words the
//      stores alone took 4000 cycles of a compute unit).  Otherwise the nodes are: lane (h, g)
//      has output column h of the nodes 8 r + 4 t + g, four codes of a code word or plane word:
//      packed words of the next layer's X, or its codes in operand order (activations between
//      the layers of a stack, see codes_offset()).
#pragma once
#include <type_traits>

#include "agg_mfma.h"
#include "layer.h"
#include "layer_parts.h"

namespace qgtc {
namespace {

// The OR over the four lane groups of eight words: lane group g keeps words 2 g and 2 g + 1.
__device__ __forceinline__ void or_reduce_8(const uint32_t (&v)[8], uint32_t (&o)[2]) {
  uint32_t r[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    // lower 32 lanes: word k of both halves, upper 32 lanes: word k + 4
    const auto q = __builtin_amdgcn_permlane32_swap(v[k], v[k + 4], false, false);
    r[k] = q[0] | q[1];
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const auto q = __builtin_amdgcn_permlane16_swap(r[k], r[k + 2], false, false);
    o[k] = q[0] | q[1];
  }
}

// Parameters of the epilogue are read from the kernel-argument segment at their point of use,
// through a pointer the compiler cannot see through: loaded at kernel entry they would sit in
// scalar registers across the aggregation and be spilled.  The lines they are in are fetched
// into the scalar cache together with the first ones (a miss costs ~800 cycles each time).
typedef const __attribute__((address_space(4))) LayerParams* LateParams;
#define QGTC_LATE(ptr) asm volatile("" : "+s"(ptr))
struct Warm {
  uint32_t v[8];
};
// Ordinary loads, one word of each line, through a pointer of their own: the compiler tracks them
// and waits in front of warm_done(), where the words are used.
__device__ __forceinline__ void warm_params(LateParams kp, Warm& w) {
  static_assert(sizeof(LayerParams) > 0x1c0 && sizeof(LayerParams) <= 0x280, "lines of 64 bytes below");
  QGTC_LATE(kp);
  const auto* words = reinterpret_cast<const __attribute__((address_space(4))) uint32_t*>(kp);
#pragma unroll
  for (int i = 0; i < 7; ++i) w.v[i] = words[16 * (i + 1)];
  w.v[7] = words[((sizeof(LayerParams) - 4) & ~63u) / 4];
}
__device__ __forceinline__ void warm_done(const Warm& w) {
  asm volatile("" :: "s"(w.v[0]), "s"(w.v[1]), "s"(w.v[2]), "s"(w.v[3]), "s"(w.v[4]), "s"(w.v[5]), "s"(w.v[6]), "s"(w.v[7]));
}

// NT = 0: one pass (at most G columns of X); the update is done output tile by output tile behind
// it.  NT > 0: several passes, the accumulators of up to NT output tiles are kept.
template <int CT, int WAYS, int NT, int SRC, int NPT, bool ROWS>
__global__ __launch_bounds__(512) void layer_kernel(const LayerParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  constexpr int G = 16 * CT * WAYS;                  // columns of a pass
  constexpr int PT = G >= 64 ? 4 : G / 16;           // 16-column tiles per column group and step of the update
  constexpr int STEPS = G > 64 ? G / 64 : 1;         // steps of the update per pass
  constexpr int OWN = 4 / WAYS;                      // tiles of the unit that the wave finishes
  constexpr int NZ = NT > 0 ? NT : 1;
  const AggParams& a = p.a;
  LateParams kp = (LateParams)__builtin_amdgcn_kernarg_segment_ptr();
  Warm warm;
  warm_params(kp, warm);
  AggWave w;
  const bool here = agg_place<WAYS, 1>(a, &w);
  warm_done(warm);
  if (!here) return;                                 // whole workgroup leaves together
  const int lane = threadIdx.x & 63;
  const int ln = lane & 15, g = lane >> 4;
  const bool self_term = a.ep.self_term != 0;
  agg_list<WAYS, 1>(a, &w, lds, self_term);

  auto mfma = [](const v4i& y, const v4i& wv, const v4i& c) {   // the update's product
    return ROWS ? __builtin_amdgcn_mfma_i32_16x16x64_i8(wv, y, c, 0, 0, 0) : __builtin_amdgcn_mfma_i32_16x16x64_i8(y, wv, c, 0, 0, 0);
  };
  const v4i zero = {0, 0, 0, 0};
  const v4i ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
  v4i z[OWN][NZ], rs[OWN];
#pragma unroll
  for (int t = 0; t < OWN; ++t) {
    rs[t] = zero;
#pragma unroll
    for (int nt = 0; nt < NZ; ++nt) z[t][nt] = zero;
  }
  uint32_t rl[OWN];                                  // per-row terms of the fp32 output

  // In front of the first loads of the aggregation: the row terms, the wave's first weights.
  // Beside them: the weights as operands (codes, minus 128 for eight bits), their column sums and the
  // column terms of the fp32 output into LDS, once per workgroup.
  uint32_t* const wsum = reinterpret_cast<uint32_t*>(lds + p.cols_off);
  double* const colterm = reinterpret_cast<double*>(lds + p.cols_off + p.n_nt_w * 64);
  const bool w8 = p.split_w != 0;
  v4u w_first = {0u, 0u, 0u, 0u}, w_first_top = {0u, 0u, 0u, 0u};
  auto before = [&]() {
    if (w.wave < p.n_nt_w) {
      const uint8_t* blk = p.wb + (int64_t)(w.wave * p.n_ks) * 1024;
      w_first = load_w<PT>(blk, lane);
      if (w8) w_first_top = load_w<PT>(blk + p.wb_part, lane);
    }
    const int32_t* row_l = p.up.row_l;
    const __amdgpu_buffer_rsrc_t rr = uniform_rsrc(row_l + w.row0, ROWS && row_l && w.rows_here > 0 ? (uint32_t)w.rows_here * 4u : 0u);
#pragma unroll
    for (int own = 0; own < OWN; ++own) {
      const int t = w.way * OWN + own;
      rl[own] = ROWS ? __builtin_amdgcn_raw_buffer_load_b32(rr, (uint32_t)(32 * (t >> 1) + 4 * (t & 1) + 8 * (ln & 3) + (ln >> 2)) * 4u, 0, 0) : 0u;
    }
  };
  auto beside = [&]() {
    LateParams k = kp;
    QGTC_LATE(k);
    const int n_nt = k->n_nt_w, n_ks = k->n_ks, w_off = k->w_off, n_out = k->h;
    const int64_t part = k->wb_part;
    const uint8_t* blk = k->wb;
    const int n_waves = k->a.n_waves;
    for (int nt = w.wave; nt < n_nt; nt += n_waves) {
      uint32_t sum = 0u;
      for (int ks = 0; ks < n_ks; ++ks) {
        v4u v = w_first, top = w_first_top;
        if (nt != w.wave || ks > 0) {
          v = load_w<PT>(blk + (int64_t)(nt * n_ks + ks) * 1024, lane);
          if (w8) top = load_w<PT>(blk + (int64_t)(nt * n_ks + ks) * 1024 + part, lane);
        }
        v |= top << 7;
#pragma unroll
        for (int i = 0; i < PT; ++i) sum = __builtin_amdgcn_sad_u8(v[i], 0u, sum);
        if (w8) v ^= 0x80808080u;
        if (w_off >= 0) *reinterpret_cast<v4u*>(lds + w_off + (ks * n_nt + nt) * 1024 + lane * 16) = v;
      }
      sum += (uint32_t)__shfl_xor((int)sum, 16, 64);
      sum += (uint32_t)__shfl_xor((int)sum, 32, 64);
      const int h = nt * 16 + ln;
      if (g == 0) wsum[h] = sum << 7;
      if (k->up.mode == QGTC_OUT_F32) {
        const int32_t* col_i = k->up.col_i;
        const double t = k->up.ck + k->up.cs * (col_i ? (double)col_i[min(h, n_out - 1)] : 0.0);
        if (g == 0) colterm[h] = t;
      }
    }
  };

  // ---- 2: the unit's codes (columns past the last one as code 0) --------------------------------
  uint8_t* const yb = lds + p.y_off + w.u * (STEPS * 64 * 16 * PT);   // [step][row in tile order][16 PT columns]
  auto write_codes = [&](LateParams k, int pass, const v4i (&acc)[4][CT], const uint32_t (&deg)[4]) {
    const Rq q = make_rq(k->a.ep.rq_lo, k->a.ep.relu, k->a.ep.rq_inv_scale, k->a.ep.rq_nbits);
    const int c0 = lane_columns<CT, PT>(w.way, g);   // the lane's columns in the pass
    const int left = k->a.cols - pass * G - c0;      // those that exist
    const uint32_t flip = k->split_y ? 0x80808080u : 0u;
    uint8_t* const to = yb + (c0 / (16 * PT)) * (64 * 16 * PT) + ln * (16 * PT) + c0 % (16 * PT);
    uint32_t keep[CT];                               // bytes of the columns that exist
#pragma unroll
    for (int ft = 0; ft < CT; ++ft) keep[ft] = (uint32_t)((1ull << (8 * min(max(left - 4 * ft, 0), 4))) - 1ull);
    constexpr int TB = 4 / CT;                       // tiles of 16 values per lane at a time
#pragma unroll
    for (int t0 = 0; t0 < 4; t0 += TB) {
      uint32_t c[4][4], d[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) c[i][r] = (uint32_t)acc[t0 + i / CT][i % CT][r] + deg[t0 + i / CT];
      pack_codes_words(c, q, d);
#pragma unroll
      for (int i = 0; i < 4; ++i) d[i] = (d[i] & keep[i % CT]) ^ flip;
      uint8_t* const at = to + t0 * (16 * 16 * PT);
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        if constexpr (CT == 4) *reinterpret_cast<v4u*>(at) = (v4u){d[0], d[1], d[2], d[3]};
        else if constexpr (CT == 2) *reinterpret_cast<v2u*>(at + t * (16 * 16 * PT)) = (v2u){d[2 * t], d[2 * t + 1]};
        else *reinterpret_cast<uint32_t*>(at + t * (16 * 16 * PT)) = d[t];
      }
    }
  };
  // codes of tile t as the operand of a step
  auto read_codes = [&](int step, int t, uint32_t flip) -> v4i {
    const uint8_t* at = yb + step * (64 * 16 * PT) + t * (16 * 16 * PT) + ln * (16 * PT) + 4 * PT * g;
    if constexpr (PT == 4) {
      return *reinterpret_cast<const v4i*>(at);
    } else if constexpr (PT == 2) {
      const v2u v = *reinterpret_cast<const v2u*>(at);
      return (v4i){(int)v.x, (int)v.y, (int)flip, (int)flip};
    } else {
      return (v4i){*reinterpret_cast<const int*>(at), (int)flip, (int)flip, (int)flip};
    }
  };

  agg_run<CT, WAYS, PT, 1, SRC, NPT>(a, w, lds, 0, self_term, before, beside, [&](int pass, const v4i (&acc)[4][CT], const uint32_t (&deg)[4]) {
    LateParams k = kp;
    QGTC_LATE(k);
    if (NT == 0) __syncthreads();                    // (the codes take the place of the slots)
    write_codes(k, pass, acc, deg);
    __syncthreads();
    if constexpr (NT > 0) {
      // ---- 3: update, all output tiles ------------------------------------------------------
      const uint32_t flip = k->split_y ? 0x80808080u : 0u;
      const int n_nt = k->n_nt_w, n_ks = k->n_ks, w_off = k->w_off;
      const bool sums = w8 || k->want_rowsum;
#pragma unroll
      for (int i = 0; i < STEPS; ++i) {
        const int ks = pass * STEPS + i;
        if (ks >= n_ks) continue;                    // (uniform)
        v4i y[OWN];
#pragma unroll
        for (int t = 0; t < OWN; ++t) y[t] = read_codes(i, w.way * OWN + t, flip);
        if (sums) {
#pragma unroll
          for (int t = 0; t < OWN; ++t) rs[t] = mfma(y[t], ones, rs[t]);
        }
        const uint8_t* blk = k->wb + (int64_t)ks * 1024;
        const int64_t nt_step = (int64_t)n_ks * 1024, part = k->wb_part;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          if (nt < n_nt) {                           // wave-uniform
            v4i wv;
            if (w_off >= 0) {
              wv = *reinterpret_cast<const v4i*>(lds + w_off + (ks * n_nt + nt) * 1024 + lane * 16);
            } else {                                 // too many for LDS
              wv = (v4i)load_w<PT>(blk + nt * nt_step, lane);
              if (w8) wv = (wv | (v4i)(load_w<PT>(blk + nt * nt_step + part, lane) << 7)) ^ (int)0x80808080;
            }
#pragma unroll
            for (int t = 0; t < OWN; ++t) z[t][nt] = mfma(y[t], wv, z[t][nt]);
          }
        }
      }
    }
  });

  // ---- 4: epilogue, 16 rows x 64 columns at a time --------------------------------------------
  // (everything it needs is read once, in front: each round of reads in the loops would cost more
  // than the arithmetic)
  LateParams k4 = kp;
  QGTC_LATE(k4);
  const bool y8 = k4->split_y != 0;
  const int mode = k4->up.mode;
  const int relu = k4->up.relu;
  const int n_out = k4->h, n_nt = k4->n_nt_w, n_ks = k4->n_ks;
  const int64_t ld_out = k4->up.ld_out, ps_out = k4->up.ps_out;
  uint8_t* const out = reinterpret_cast<uint8_t*>(k4->up.out);
  const float* const col_a = k4->up.col_a;
  const float* const col_b = k4->up.col_b;
  const Rq q = make_rq(k4->up.rq_lo, relu, k4->up.rq_inv_scale, k4->up.rq_nbits);
  const uint32_t oflip = k4->up.rq_nbits == 8 ? 0x80808080u : 0u;
  const bool want_rowsum = k4->want_rowsum != 0, sums = w8 || want_rowsum;
  const double cc = k4->up.cc, l0a = k4->up.l0a, l0b = k4->up.l0b, rsc = k4->up.rs;
  const int32_t* const row_i = k4->up.row_i;
  const uint8_t* const wl = lds + k4->w_off + lane * 16;
  // the packed words of the unit [half][plane][column], put together in LDS by its waves
  uint32_t* const planes = reinterpret_cast<uint32_t*>(lds + k4->planes_off) + w.u * 16 * n_out;
  if (!ROWS && mode == QGTC_OUT_BITS) {
    if (NT > 0) __syncthreads();                     // every wave is through with the slots
    for (int i = w.way * 64 + lane; i < 16 * n_out; i += 64 * WAYS) planes[i] = 0u;
    __syncthreads();
  }
  const uint32_t ld4 = (uint32_t)ld_out * 4u;
  const uint32_t flip = y8 ? 0x80808080u : 0u;
  // (the wave's tiles go through each step together: chains of reads and products overlap)
  v4i y[OWN][STEPS], rowadd[OWN];
  double t1[OWN], l0[OWN];
  __amdgpu_buffer_rsrc_t ro[OWN];
  int t[OWN], row32[OWN], rows_here[OWN];
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    const int ut = w.way * OWN + o;                  // tile of the unit
    t[o] = ut & 1;
    row32[o] = w.row0 + 32 * (ut >> 1);
    rows_here[o] = max(min(w.rows_here - 32 * (ut >> 1), 32), 0);
    if constexpr (NT == 0) {
      rs[o] = zero;
#pragma unroll
      for (int i = 0; i < STEPS; ++i) y[o][i] = read_codes(i, ut, flip);
    }
  }
  if (NT == 0 && sums) {
#pragma unroll
    for (int o = 0; o < OWN; ++o)
#pragma unroll
      for (int i = 0; i < STEPS; ++i)
        if (i < n_ks) rs[o] = mfma(y[o][i], ones, rs[o]);
  }
#pragma unroll
  for (int o = 0; o < OWN; ++o) {
    t1[o] = l0[o] = 0.0;
    if (ROWS && mode == QGTC_OUT_F32) {
      // this lane's node: a sum of codes (unsigned), or the caller's int32
      double ri = 0.0;
      if (want_rowsum) ri = (double)((uint32_t)rs[o][0] + (y8 ? (uint32_t)(n_ks * 64) << 7 : 0u));
      else if (row_i) ri = (double)row_i[min(row32[o] + 8 * (ln & 3) + 4 * t[o] + (ln >> 2), k4->a.rows - 1)];
      t1[o] = rsc * ri;
      l0[o] = l0a + l0b * (double)(int32_t)rl[o];
    }
    rowadd[o] = w8 ? rs[o] << 7 : zero;
    // the 32 rows as one buffer; rows past the last one fall outside
    ro[o] = uniform_rsrc(out + (ROWS ? (int64_t)row32[o] * ld_out * 4 : 0),
                         rows_here[o] > 0 ? (uint32_t)(rows_here[o] - 1) * ld4 + (uint32_t)n_out * 4u : 0u);
  }
  constexpr int NB = NT == 1 ? 1 : (OWN == 4 ? 2 : 4);   // output tiles side by side
#pragma unroll 1
  for (int nt0 = 0; nt0 < n_nt; nt0 += NB) {
    v4i zz[OWN][NB];
    int at[NB];                                      // (the last tile again in place of those past it)
#pragma unroll
    for (int j = 0; j < NB; ++j) at[j] = min(nt0 + j, n_nt - 1) * 16;
    if constexpr (NT == 0) {
      // ---- 3: update of these tiles ----------------------------------------------------------
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
          if (i >= n_ks) continue;
          const v4i wv = *reinterpret_cast<const v4i*>(wl + i * n_nt * 1024 + at[j] * 64);
#pragma unroll
          for (int o = 0; o < OWN; ++o) zz[o][j] = mfma(y[o][i], wv, i == 0 ? rowadd[o] : zz[o][j]);
        }
    } else {
#pragma unroll
      for (int o = 0; o < OWN; ++o) {
#pragma unroll
        for (int j = 0; j < NB; ++j) zz[o][j] = z[o][j] + rowadd[o];
#pragma unroll
        for (int k = 0; k + NB < NZ; ++k) z[o][k] = z[o][k + NB];   // the next tiles move to the front
      }
    }
    if (y8) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        v4i add;
        if (ROWS) {
          add = *reinterpret_cast<const v4i*>(wsum + at[j] + 4 * g);
        } else {
          const int c = (int)wsum[at[j] + ln];
          add = (v4i){c, c, c, c};
        }
#pragma unroll
        for (int o = 0; o < OWN; ++o) zz[o][j] += add;
      }
    }
    if constexpr (ROWS) {
      v4u res[OWN][NB];
      if (mode == QGTC_OUT_I32) {
#pragma unroll
        for (int o = 0; o < OWN; ++o)
#pragma unroll
          for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) res[o][j][r] = (uint32_t)(relu ? max(zz[o][j][r], 0) : zz[o][j][r]);
      } else {
        // the arithmetic of dequantize_f64, with the row and column terms formed once
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          double ct[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) ct[r] = colterm[at[j] + 4 * g + r];
          double ca[4], cb[4];
          if (col_a) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int hc = min(at[j] + 4 * g + r, n_out - 1);
              ca[r] = (double)col_a[hc];
              cb[r] = col_b ? (double)col_b[hc] : 0.0;
            }
          }
#pragma unroll
          for (int o = 0; o < OWN; ++o)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              double v = (cc * (double)zz[o][j][r] + t1[o]) + l0[o] * ct[r];
              if (col_a) v = v * ca[r] + cb[r];
              if (relu) v = v < 0.0 ? 0.0 : v;
              res[o][j][r] = __float_as_uint((float)v);
            }
        }
      }
#pragma unroll
      for (int o = 0; o < OWN; ++o) {
        const int node = 8 * (ln & 3) + 4 * t[o] + (ln >> 2);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          if (nt0 + j >= n_nt) continue;             // wave-uniform
          const int h = at[j] + 4 * g;
          if (ld_out < (1 << 22)) {                  // 32 rows within 2^29 bytes: offsets below the one of no store
            const uint32_t off = (uint32_t)node * ld4 + (uint32_t)h * 4u;
            if (h + 4 <= n_out) {
              __builtin_amdgcn_raw_buffer_store_b128(res[o][j], ro[o], off, 0, 0);
            } else {
#pragma unroll
              for (int r = 0; r < 4; ++r)
                __builtin_amdgcn_raw_buffer_store_b32(res[o][j][r], ro[o], h + r < n_out ? off + 4u * r : 0xc0000000u, 0, 0);
            }
          } else if (node < rows_here[o]) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (h + r < n_out) reinterpret_cast<uint32_t*>(out)[(row32[o] + node) * ld_out + h + r] = res[o][j][r];
          }
        }
      }
    } else {
#pragma unroll
      for (int o = 0; o < OWN; ++o) {
        if (rows_here[o] <= 0) continue;             // wave-uniform
        uint32_t c[NB];
        if (col_a) {
          const uint32_t qmax = (uint32_t)q.qmaxf;
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const int hc = min(at[j] + ln, n_out - 1);
            const float ca = col_a[hc], cb = col_b ? col_b[hc] : 0.0f;
            c[j] = 0u;
#pragma unroll
            for (int r = 0; r < 4; ++r)
              c[j] |= requantize_affine((uint32_t)zz[o][j][r], ca, cb, relu, q.lo, q.inv, qmax, q.qmaxf) << (8 * r);
          }
        } else {
          uint32_t cz[4][4], cw[4];
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) cz[j][r] = (uint32_t)zz[o][j % NB][r];
          pack_codes_words(cz, q, cw);
#pragma unroll
          for (int j = 0; j < NB; ++j) c[j] = cw[j];
        }
        if (rows_here[o] < 32) {                     // bytes of the rows that exist
          const uint32_t m = (uint32_t)((1ull << (8 * min(max((rows_here[o] - (4 * t[o] + g) + 7) >> 3, 0), 4))) - 1ull);
#pragma unroll
          for (int j = 0; j < NB; ++j) c[j] &= m;
        }
        if (mode == kOutCodes) {
          // code word 4 t + g of this column and word row; ld_out: log2 of the column tiles per group
          const int l = (int)ld_out;
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if (nt0 + j >= n_nt) continue;           // wave-uniform
            const int h = at[j] + ln, k = h & ((16 << l) - 1);
            const int pos = 16 * ((k >> 2) & ((1 << l) - 1)) + 4 * (k >> (2 + l)) + (k & 3);
            uint8_t* dst = out + (int64_t)(h >> (4 + l)) * ps_out + (((int64_t)(row32[o] >> 5) * 512 + 256 * t[o]) << l) + pos * 16 + 4 * g;
            *reinterpret_cast<uint32_t*>(dst) = c[j] ^ oflip;
          }
        } else {
          const int half = (w.way * OWN + o) >> 1;
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if (nt0 + j >= n_nt) continue;           // wave-uniform
            // planes: this lane's bits are 8 r + 4 t + g of the word
            uint32_t v[8], ow[2];
#pragma unroll
            for (int pl = 0; pl < 8; ++pl) v[pl] = ((c[j] >> pl) & 0x01010101u) << (4 * t[o] + g);
            or_reduce_8(v, ow);
            const int h = at[j] + ln;
            if (h < n_out) {
              atomicOr(&planes[(8 * half + 2 * g) * n_out + h], ow[0]);
              atomicOr(&planes[(8 * half + 2 * g + 1) * n_out + h], ow[1]);
            }
          }
        }
      }
    }
  }
  if (!ROWS && mode == QGTC_OUT_BITS) {
    __syncthreads();
    const int qbits = k4->up.rq_nbits;
    for (int half = 0; half < 2; ++half) {
      if (w.rows_here <= 32 * half) break;
      uint32_t* words = reinterpret_cast<uint32_t*>(out) + (int64_t)((w.row0 >> 5) + half) * ld_out;
      for (int h = w.way * 64 + lane; h < n_out; h += 64 * WAYS)
        for (int pl = 0; pl < qbits; ++pl) words[(int64_t)pl * ps_out + h] = planes[(8 * half + pl) * n_out + h];
    }
  }
}

template <int CT, int WAYS, int NT, int SRC, int NPT, bool ROWS>
qgtc_status launch_one(const LayerParams& p, size_t lds, hipStream_t stream) {
  static OncePerDevice once;
  if (!allow_lds(once, reinterpret_cast<const void*>(&layer_kernel<CT, WAYS, NT, SRC, NPT, ROWS>), lds)) return QGTC_ERR_HIP;
  hipLaunchKernelGGL((layer_kernel<CT, WAYS, NT, SRC, NPT, ROWS>), dim3(xcd_deal_grid(p.a.nblocks, p.a.run_shift)),
                     dim3((unsigned)(64 * p.a.n_waves)), lds, stream, p);
  return launch_status();
}

template <int CT, int WAYS, int NT, int SRC, int NPT>
qgtc_status launch_mode(const LayerParams& p, size_t lds, hipStream_t stream) {
  const bool rows = p.up.mode == QGTC_OUT_I32 || p.up.mode == QGTC_OUT_F32;
  return rows ? launch_one<CT, WAYS, NT, SRC, NPT, true>(p, lds, stream) : launch_one<CT, WAYS, NT, SRC, NPT, false>(p, lds, stream);
}

template <int CT, int WAYS, int NT>
qgtc_status launch_src(const LayerParams& p, bool codes, size_t lds, hipStream_t stream) {
  if (codes) return launch_mode<CT, WAYS, NT, kSrcCodes, 1>(p, lds, stream);
  switch (agg_items_per_thread(p.a, AggSplit{CT, WAYS, 0, 1})) {
    case 1: return launch_mode<CT, WAYS, NT, kSrcPlanes, 1>(p, lds, stream);
    case 2: return launch_mode<CT, WAYS, NT, kSrcPlanes, 2>(p, lds, stream);
    default: return launch_mode<CT, WAYS, NT, kSrcPlanes, 4>(p, lds, stream);
  }
}

}  // namespace

template <int NT>
qgtc_status layer_launch(const LayerParams& p, const AggSplit& sp, bool codes, size_t lds, hipStream_t stream) {
  if constexpr (NT == 0) {
    switch (8 * sp.ct + sp.ways) {
      case 8 * 1 + 1: return launch_src<1, 1, NT>(p, codes, lds, stream);
      case 8 * 1 + 2: return launch_src<1, 2, NT>(p, codes, lds, stream);
      case 8 * 1 + 4: return launch_src<1, 4, NT>(p, codes, lds, stream);
      case 8 * 2 + 2: return launch_src<2, 2, NT>(p, codes, lds, stream);
    }
  }
  if constexpr (NT < 16)
    if (sp.ct == 4) return launch_src<4, 2, NT>(p, codes, lds, stream);
  return launch_src<2, 4, NT>(p, codes, lds, stream);
}

}  // namespace qgtc
