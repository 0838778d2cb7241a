// Neighbour aggregation C = A.X by itself (first half of Algorithm 1; zero-tile jumping and
// non-zero tile reuse, Sections 4.3 and 4.4 of the paper): the product of agg_mfma.h with
// the output epilogues.  X of more than eight planes is taken eight planes at a time and
// the partial results are shifted and added (modulo 2^32).
#include "agg_dense.h"

namespace qgtc {
namespace {

// Bytes of a column group of codes.
int64_t codes_group_bytes(int kwords, int lt) { return (int64_t)kwords * 512 * lt; }

struct CodesParams {
  const uint32_t* X;
  int64_t ld, ps;
  int32_t s, cols, kwords;
  uint8_t* dst;
  int64_t cg_bytes;          // of a column group
  uint32_t flip;
};

// Planes to codes in the staged order of agg_run(): a thread has 32 rows of a column.  Bound by its launch
// (16384 x 256 of 4 bits: 2 MB in, 4 MB out).
template <int LT>
__global__ __launch_bounds__(256) void planes_to_codes_kernel(const CodesParams p) {
  constexpr int G = 16 * LT, KB = 512 * LT;
  const unsigned idx = blockIdx.x * 256u + threadIdx.x, cg = blockIdx.y;
  const int kw = (int)(idx / G), c = (int)(idx % G);
  if (kw >= p.kwords) return;
  const uint32_t* const from = p.X + (int64_t)kw * p.ld + min((int)cg * G + c, p.cols - 1);
  uint32_t a[8];
#pragma unroll
  for (int pl = 0; pl < 8; ++pl) {
    a[pl] = 0u;
    if (pl < p.s) a[pl] = from[(int64_t)pl * p.ps];
  }
  planes_word_to_codes(a);
  uint8_t* const to = p.dst + (int64_t)cg * p.cg_bytes + (int64_t)kw * KB + staged_pos<LT>(c) * 16;
  *reinterpret_cast<v4u*>(to) = (v4u){a[0], a[1], a[2], a[3]} ^ p.flip;
  *reinterpret_cast<v4u*>(to + LT * 256) = (v4u){a[4], a[5], a[6], a[7]} ^ p.flip;
}

template <int CT, int WAYS, int KS, int SRC, int NPT, bool MULTI>
__global__ __launch_bounds__(512) void aggregate_kernel(const AggParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  constexpr int LC = 4 * CT;                         // columns of a lane
  AggWave w;
  if (!agg_place<WAYS, KS>(p, &w)) return;               // whole workgroup leaves together
  const int lane = threadIdx.x & 63;
  const int ln = lane & 15, g = lane >> 4;
  const EpiParams& e = p.ep;
  const bool self_term = e.self_term != 0;
  const int cg = w.cw * WAYS + w.way, last_cg = (p.cols - 1) / (16 * CT);
  agg_list<WAYS, KS>(p, &w, lds, self_term);

  uint32_t y[4][LC];
  for (int plane0 = 0; plane0 < (MULTI ? p.s : 1); plane0 += 8) {
    if (MULTI && plane0 > 0) __syncthreads();        // every wave is through with the slots
    agg_run<CT, WAYS, CT, KS, SRC, NPT>(p, w, lds, plane0, self_term, [] {}, [] {},
                                       [&](int, const v4i (&acc)[4][CT], const uint32_t (&deg)[4]) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int ft = 0; ft < CT; ++ft)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint32_t v = (uint32_t)acc[t][ft][r] + deg[t];
            if (MULTI && plane0 > 0) y[t][4 * ft + r] += v << plane0;
            else y[t][4 * ft + r] = v;
          }
    });
  }

  // The waves of a unit that had parts of the stages add up, and finish one tile each.
  int tile_from = 0, tile_to = 4;
  if constexpr (KS > 1) {
    static_assert(KS == 4, "a tile per wave");
    __syncthreads();                                 // every wave is through with the slots
    uint32_t* box = reinterpret_cast<uint32_t*>(lds) + lane;
    constexpr int BOX = 4 * LC * 64;                 // words of a wave: [tile][column][lane]
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int k = 0; k < LC; ++k) box[w.wave * BOX + (t * LC + k) * 64] = y[t][k];
    __syncthreads();
    const int first = w.wave - w.kp * WAYS;
#pragma unroll
    for (int k = 0; k < LC; ++k) {
      uint32_t v = 0u;
#pragma unroll
      for (int j = 0; j < KS; ++j) v += box[(first + j * WAYS) * BOX + (w.kp * LC + k) * 64];
      y[0][k] = v;
    }
    tile_from = w.kp;
    tile_to = w.kp + 1;
  }
  if (cg > last_cg || w.rows_here <= 0) return;      // no barrier follows

  auto next_tile = [&]() {
#pragma unroll
    for (int k = 0; k < LC; ++k) {
      y[0][k] = y[1][k];
      y[1][k] = y[2][k];
      y[2][k] = y[3][k];
    }
  };

  // lane (n, g): columns col0 .. col0 + LC - 1 of row n of its tile
  auto row_of = [&](int tile) { return 32 * (tile >> 1) + 8 * (ln & 3) + 4 * (tile & 1) + (ln >> 2); };
  const int col0 = cg * 16 * CT + LC * g;
  if (e.mode == QGTC_OUT_I32 || e.mode == QGTC_OUT_F32) {
    const bool vec = (e.ld_out & 3) == 0 && ((uintptr_t)e.out & 15u) == 0;   // 16-byte stores
#pragma unroll 1
    for (int tile = tile_from; tile < tile_to; ++tile) {
      if (tile > tile_from) next_tile();
      constexpr int t = 0;                           // (the current tile is in front)
      const int j = row_of(tile), row = w.row0 + j;
      if (j >= w.rows_here) continue;
      uint32_t o[LC];
      if (e.mode == QGTC_OUT_I32) {
#pragma unroll
        for (int k = 0; k < LC; ++k) o[k] = (e.relu && (int32_t)y[t][k] < 0) ? 0u : y[t][k];
      } else {
        // the arithmetic of dequantize_f64, with the row terms formed once
        const double ri = e.row_i ? (double)e.row_i[row] : 0.0;
        const double l0 = e.l0a + e.l0b * (e.row_l ? (double)e.row_l[row] : 0.0);
#pragma unroll
        for (int k = 0; k < LC; ++k) {
          const int cc = min(col0 + k, p.cols - 1);
          const double t1 = e.cc * (double)(int32_t)y[t][k] + e.rs * ri;
          double v = t1 + l0 * (e.ck + e.cs * (e.col_i ? (double)e.col_i[cc] : 0.0));
          if (e.col_a) v = v * (double)e.col_a[cc] + (e.col_b ? (double)e.col_b[cc] : 0.0);
          if (e.relu && v < 0.0) v = 0.0;
          o[k] = __float_as_uint((float)v);
        }
      }
      uint32_t* dst = reinterpret_cast<uint32_t*>(e.out) + (int64_t)row * e.ld_out + col0;
#pragma unroll
      for (int k = 0; k < LC; k += 4) {
        if (vec && col0 + k + 4 <= p.cols) {
          *reinterpret_cast<v4u*>(dst + k) = (v4u){o[k], o[k + 1], o[k + 2], o[k + 3]};
        } else {
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (col0 + k + q < p.cols) dst[k + q] = o[k + q];
        }
      }
    }
    return;
  }

  // Packed planes along the columns: the lane's codes are 4 or 8 consecutive bits of a
  // word; it stores bytes or 16-bit halves where that is a whole number of bytes.
  const int qbits = e.rq_nbits;
  const uint32_t qmax = qbits >= 32 ? 0xffffffffu : ((1u << qbits) - 1u);
  const float qmaxf = (float)qmax;
  const int data_words = (p.cols + 31) >> 5;
#pragma unroll 1
  for (int tile = tile_from; tile < tile_to; ++tile) {
    if (tile > tile_from) next_tile();
    constexpr int t = 0;
    const int j = row_of(tile), row = w.row0 + j;
    const bool row_ok = j < w.rows_here;
#pragma unroll
    for (int k = 0; k < LC; ++k)
      y[t][k] = col0 + k < p.cols ? requantize_i32(y[t][k], min(col0 + k, p.cols - 1), e, qmax, qmaxf) : 0u;
    uint32_t* drow = reinterpret_cast<uint32_t*>(e.out) + (int64_t)(row_ok ? row : 0) * e.ld_out;
    for (int p0 = 0; p0 < qbits; p0 += 8) {
      // 8 x 8 bit transposes: byte i of (lo, hi) holds bit p0 + i of eight codes
      uint32_t lo[(LC + 7) / 8], hi[(LC + 7) / 8];
#pragma unroll
      for (int b = 0; b < (LC + 7) / 8; ++b) {
        lo[b] = hi[b] = 0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (8 * b + k >= LC) continue;
          const uint32_t c = (y[t][8 * b + k] >> p0) & 0xffu;
          if (k < 4) lo[b] |= c << (8 * k);
          else hi[b] |= c << (8 * (k - 4));
        }
        transpose_bits_8x8(lo[b], hi[b]);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int sh = 8 * (i & 3);
        uint32_t v[(LC + 7) / 8];
#pragma unroll
        for (int b = 0; b < (LC + 7) / 8; ++b) v[b] = ((i < 4 ? lo[b] : hi[b]) >> sh) & 0xffu;
        uint32_t* dst = drow + (int64_t)(p0 + i) * e.ps_out;
        const bool plane_ok = p0 + i < qbits;
        if constexpr (CT == 2) {
          if (plane_ok && row_ok) reinterpret_cast<uint8_t*>(dst)[4 * cg + g] = (uint8_t)v[0];
        } else {
          uint32_t word = v[0] << (4 * g);
          word |= (uint32_t)__shfl_xor((int)word, 16, 64);
          word |= (uint32_t)__shfl_xor((int)word, 32, 64);
          if (plane_ok && row_ok && g == 0) {
            if ((cg & 1) == 0 && cg == last_cg) dst[cg >> 1] = word;   // nothing in the upper half
            else reinterpret_cast<uint16_t*>(dst)[cg] = (uint16_t)word;
          }
        }
      }
    }
    // a LEFT operand has zeros between the last data word of a row and its leading dimension
    if (cg == last_cg && row_ok) {
      for (int pl = 0; pl < qbits; ++pl)
        for (int wd = data_words + g; wd < (int)e.ld_out; wd += 4) drow[(int64_t)pl * e.ps_out + wd] = 0u;
    }
  }
}

template <int CT, int WAYS, int KS, int SRC, int NPT, bool MULTI>
qgtc_status launch_one(const AggParams& p, size_t lds, hipStream_t stream) {
  static OncePerDevice once;
  if (!allow_lds(once, reinterpret_cast<const void*>(&aggregate_kernel<CT, WAYS, KS, SRC, NPT, MULTI>), lds)) return QGTC_ERR_HIP;
  hipLaunchKernelGGL((aggregate_kernel<CT, WAYS, KS, SRC, NPT, MULTI>), dim3(xcd_deal_grid(p.nblocks, p.run_shift)),
                     dim3((unsigned)(64 * p.n_waves)), lds, stream, p);
  return launch_status();
}

template <int CT, int WAYS, int KS>
qgtc_status launch(const AggParams& p, size_t lds, hipStream_t stream) {
  const bool multi = p.s > 8;
  switch (agg_items_per_thread(p, AggSplit{CT, WAYS, CT, KS})) {
    case 1: return multi ? launch_one<CT, WAYS, KS, kSrcPlanes, 1, true>(p, lds, stream) : launch_one<CT, WAYS, KS, kSrcPlanes, 1, false>(p, lds, stream);
    case 2: return multi ? launch_one<CT, WAYS, KS, kSrcPlanes, 2, true>(p, lds, stream) : launch_one<CT, WAYS, KS, kSrcPlanes, 2, false>(p, lds, stream);
    default: return multi ? launch_one<CT, WAYS, KS, kSrcPlanes, 4, true>(p, lds, stream) : launch_one<CT, WAYS, KS, kSrcPlanes, 4, false>(p, lds, stream);
  }
}

// From codes, which are made first.
template <int CT, int WAYS, int KS>
qgtc_status launch_codes(AggParams* p, const qgtc_bits* X, void* workspace, size_t lds, hipStream_t stream) {
  CodesParams c{};
  c.X = X->data;
  c.ld = X->ld_words;
  c.ps = X->plane_stride_words;
  c.s = X->nbits;
  c.cols = X->cols;
  c.kwords = p->x_kwords;
  c.dst = reinterpret_cast<uint8_t*>(workspace);
  c.cg_bytes = codes_group_bytes(p->x_kwords, CT);
  c.flip = X->nbits == 8 ? 0x80808080u : 0u;
  hipLaunchKernelGGL(planes_to_codes_kernel<CT>, dim3((unsigned)cdiv((int64_t)c.kwords * 16 * CT, 256), (unsigned)cdiv(c.cols, 16 * CT)), dim3(256),
                     0, stream, c);
  const qgtc_status st = launch_status();
  if (st != QGTC_OK) return st;
  p->X = reinterpret_cast<const uint32_t*>(workspace);
  p->x_bytes = (uint32_t)c.cg_bytes;
  return launch_one<CT, WAYS, KS, kSrcCodes, 1, false>(*p, lds, stream);
}

}  // namespace

// Narrower column groups where wide ones would leave compute units without a workgroup of two
// units: the rows of A are then expanded once per group, which costs less than idle units.
// Where that leaves two or fewer waves per compute unit, four of them share a unit's stages
// (8192 x 8192 x 64: two waves of 16 columns 33 us, eight of them 18 us), unless all of K is one
// stage of two chunks anyway (1024 x 1024 x 64: four stages 8.6 us, one for all waves 4.7 us).  With
// up to four waves per compute unit it depends on the adjacency: every tile occupied 8192 x 8192 x
// 128 36.5 and 33.4 us, diagonal blocks of 256 in 4096 x 4096 x 200 7.3 and 11.5 us.
AggSplit aggregate_split(int rows, int cols, int a_words, int64_t lda) {
  const int64_t units = cdiv(rows, kUnitRows), enough = 2 * (int64_t)device_compute_units();
  AggSplit sp{2, 2, 2, 1};
  if (cols <= 32 || units * cdiv(cols, 64) < enough) sp = AggSplit{1, 2, 1, 1};
  if (agg_long_rows(lda)) return sp;
  if (cols <= 16 || units * cdiv(cols, 32) < enough) sp = AggSplit{1, 1, 1, units * cdiv(cols, 16) <= enough && a_words > 8 ? 4 : 1};
  return sp;
}

}  // namespace qgtc

using namespace qgtc;

extern "C" int32_t qgtc_aggregate_reads_map(const qgtc_bits* A, int32_t x_cols) {
  AggParams p{};
  if (!A || x_cols < 1 || agg_fill_adjacency(A, nullptr, &p) != QGTC_OK || A->rows == 0) return 0;
  p.cols = x_cols;
  const AggSplit sp = aggregate_split(A->rows, x_cols, p.a_words, A->ld_words);
  (void)agg_set_shape(&p, sp, cdiv(x_cols, sp.group()), 0);
  return agg_reads_map(p, sp) ? 1 : 0;
}

// A codes' column group is addressed with 32 bits; features of more codes stay as planes.
constexpr int64_t kMostCodes = (int64_t)256 << 20;
static int64_t codes_bytes(const AggParams& p, const AggSplit& sp) { return codes_group_bytes(p.x_kwords, sp.lt) * cdiv(p.cols, 16 * sp.lt); }

// Whether the features are turned into codes by a launch of their own (3 us) instead of by every workgroup, for
// whom a stage of planes goes through registers, whose wait is also one for the stage's words of A: from
// nine stages of K on.  Planes and codes as bytes, us:
//   stages of two chunks: 2048 rows per block (eight stages), 64 columns 19.1 and 17.8, 128 columns 22.8 and 24.2;
//   3072 x 256 (twelve) 19.8 and 17.8; 8192 x 300 71 and 51; 16384 x 256 112 and 90
//   of eight, which four waves share: 4096 x 64 (four) 10.4 and 10.7; 8192 x 64 (eight) 18.9 and 18.7, and with
//   the launch from a script 17.1 and 17.5; 12288 x 16 (twelve) 22.4 and 17.8; 256 x 65536 x 64 94 and 65
static bool aggregate_from_codes(const AggParams& p, const AggSplit& sp) {
  return p.s <= 8 && p.a_words > 32 * sp.chunks() && codes_bytes(p, sp) <= kMostCodes;
}

// Whether they become operands of 4- or 6-bit floats (agg_dense.hip) instead, where the sums are exact there.  odd: rows of
// the output that are not whole 16 bytes.  Measured over 300 drawn shapes of 200 to 60000 rows, 2100 to 30000 columns of A and 4 to
// 600 of X, every tile occupied; bytes (or planes) and floats, us:
//   1 to 4 bits, one product per word: from nine stages on wherever rows fill the chip with undivided stages (16384 x 16384 x 256 at
//   4 bits 89 and 46, 16400 x 2500 x 64 15.6 and 12.5).  Diagonal blocks of up to 3072 rows that are more than two rounds of
//   workgroups are not: X is as long as A and its operands are written once more (81920 x 256 at 4 bits 102 and 119).
//   Where four waves share a unit's stages, 1 and 2 bits and up to 32 columns of 3 and 4 as before (1161 x 21479 x 32 23.7 and
//   17.1), wider rows of 3 and 4 bits where workgroups of 32 rows and 64 columns fill half of the chip (7889 x 15121 x 47
//   24.1 and 21.2; 1350 x 6699 x 46, 43 workgroups, 12.8 and 13.7).  That many have floats earlier too, of more than 4608
//   columns of A instead of 8192 (5000 x 5000 x 64 at 2 bits 12.5 and 10.1; 1603 x 4608 x 58 10.1 and 10.4), and up to 32
//   columns of 1024 rows and more from 7168 (1024 x 7200 x 32 13.4 and 10.4).
//   5 to 8 bits, two products per word and 32 columns per workgroup: undivided stages in one round of workgroups (16384 x 16384 x 64 at 8
//   55.6 and 30.1; 13932 x 2760 x 384, 2.6 rounds, 44.6 and 53.9), with odd rows, whose stores cost bytes more (16551 x 3077 x 574,
//   4.6 rounds, 124 and 101), or of more than 10240 columns without a map (16384 x 16384 x 256 90 and 78; with one of blocks of 256
//   17815 x 17815 x 556 38.8 and 78.9).  Divided ones up to 64 columns (with a launch beside them, as it is used: 10507 x 10507 x 24
//   27.4 and 25.1, 16384 x 16384 x 32 34.7 and 31.2, 1000 x 9000 x 64 22.5 and 20.8, 300 x 30000 x 50 40.6 and 37.2; 5000 x 9000 x 40 22.8 and
//   23.4; a map of blocks of 4096 9500 x 9500 x 32 21.1 and 21.4, 8300 x 8300 x 17 20.4 and 22.3), not more (461 x 8274 x 433 15.5 and 20.6).
//   Not 16 or fewer columns, half of whose tiles of 32 would be empty (12288 x 12288 x 16 17.9 and 20.1).
// With a map that leaves most tiles out floats lose some: the launch in front, and more rows per list (8192 x 8192 x 64 at 2
// bits with eight full blocks on the diagonal 6.9 and 9.2, sixteen in 16384 x 16384 x 256 at 4 19.1 and 21.0; with every
// tile 15.6 and 11.8, 89 and 46).  How full a map is only the device knows.
static bool aggregate_from_floats(const AggParams& p, const AggSplit& sp, bool odd) {
  if (!dense_applies(p) || codes_bytes(p, sp) > kMostCodes || (p.cols <= 16 && p.s > 4)) return false;
  const bool long_rows = p.a_words > 32 * sp.chunks();
  const int64_t cus = device_compute_units();
  if (sp.ks == 1) {
    if (!long_rows) return false;
    const int64_t rounds = cdiv(dense_groups(p, 256), cus);
    return p.s > 4 ? rounds == 1 || odd || (!p.row_cnt && p.a_words > 320) : !(p.block_rows > 0 && p.a_words <= 96 && rounds > 2);
  }
  if (p.s > 4) return long_rows && p.cols <= 64;
  if (p.cols <= 32) return long_rows || (p.rows >= 1024 && p.a_words > 224);
  const bool many = dense_groups(p, 32) > cus / 2;
  return (long_rows && (many || p.s <= 2)) || (many && p.a_words > 144);
}

extern "C" size_t qgtc_aggregate_workspace_bytes(const qgtc_bits* A, const qgtc_bits* X) {
  AggParams p{};
  if (!A || !X || A->rows == 0 || X->cols == 0 || agg_fill_params(A, nullptr, X, &p) != QGTC_OK) return 0;
  const AggSplit sp = aggregate_split(A->rows, X->cols, p.a_words, A->ld_words);
  // (where the output decides, bytes need less)
  if (aggregate_from_floats(p, sp, true)) return (size_t)dense_bytes(p);
  return aggregate_from_codes(p, sp) ? (size_t)codes_bytes(p, sp) : 0;
}

extern "C" qgtc_status qgtc_aggregate_ws(const qgtc_bits* A, const qgtc_tile_map* map, const qgtc_bits* X,
                                         const qgtc_epilogue* ep, void* workspace, size_t workspace_bytes, void* out,
                                         int64_t ld_out, void* stream) {
  if (!A || !X || !ep) return QGTC_ERR_NULL;
  AggParams p{};
  qgtc_status st = agg_fill_params(A, map, X, &p);
  if (st != QGTC_OK) return st;
  if (!out) return (A->rows == 0 || X->cols == 0) ? QGTC_OK : QGTC_ERR_NULL;   // an empty result needs no buffer
  const bool square = A->block_rows > 0 || A->rows == A->cols;
  st = make_epilogue(ep, out, ld_out, A->rows, X->cols, QGTC_LEFT, square, &p.ep);
  if (st != QGTC_OK) return st;
  st = check_tuning(ep->tuning);
  if (st != QGTC_OK) return st;
  if (A->rows == 0 || X->cols == 0) return QGTC_OK;

  const AggSplit sp = aggregate_split(A->rows, X->cols, p.a_words, A->ld_words);
  const size_t lds = agg_set_shape(&p, sp, cdiv(X->cols, sp.group()), ep->tuning ? ep->tuning->agg_xcd_run : 0);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope prof(QGTC_KERNEL_AGGREGATE, s);
  // (room that is no room for floats may still be enough for bytes, and is not needed for planes)
  const bool odd = ep->mode != QGTC_OUT_BITS && ((ld_out & 3) != 0 || ((uintptr_t)out & 15u) != 0);
  if (workspace && aggregate_from_floats(p, sp, odd) && ((uintptr_t)workspace & 15u) == 0 && workspace_bytes >= (size_t)dense_bytes(p))
    return dense_aggregate(p, workspace, ep->tuning ? ep->tuning->agg_xcd_run : 0, s);
  if (workspace && aggregate_from_codes(p, sp)) {
    if (((uintptr_t)workspace & 15u) != 0) return QGTC_ERR_ALIGN;
    if (workspace_bytes < (size_t)codes_bytes(p, sp)) return QGTC_ERR_WORKSPACE;
    if (sp.ct == 2) return launch_codes<2, 2, 1>(&p, X, workspace, lds, s);
    if (sp.ways == 2) return launch_codes<1, 2, 1>(&p, X, workspace, lds, s);
    return sp.ks == 4 ? launch_codes<1, 1, 4>(&p, X, workspace, lds, s) : launch_codes<1, 1, 1>(&p, X, workspace, lds, s);
  }
  if (sp.ct == 2) return launch<2, 2, 1>(p, lds, s);
  if (sp.ways == 2) return launch<1, 2, 1>(p, lds, s);
  return sp.ks == 4 ? launch<1, 1, 4>(p, lds, s) : launch<1, 1, 1>(p, lds, s);
}

extern "C" qgtc_status qgtc_aggregate(const qgtc_bits* A, const qgtc_tile_map* map, const qgtc_bits* X,
                                      const qgtc_epilogue* ep, void* out, int64_t ld_out, void* stream) {
  return qgtc_aggregate_ws(A, map, X, ep, nullptr, 0, out, ld_out, stream);
}
