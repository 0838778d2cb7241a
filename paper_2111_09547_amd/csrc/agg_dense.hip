// Aggregation of long rows, C = A.X with A binary and X of at most 8 bits, on v_mfma_scale_f32_32x32x64_f8f6f4.
//
// The instruction takes 4-bit (E2M1) and 6-bit (E2M3) floats at twice the rate of bytes (8.2 to 9.6 against
// 3.5 to 4.2 POP/s from registers, four sums per wave), and small integers are exact in both, as are fp32 sums below 2^24, which the rule in
// dense_applies() keeps to.  What it saves more of is the way there:
//   A  a word w of 32 bits is the 4-bit operand after five instructions instead of fifteen and in half the
//      registers: w & 0x11111111, w & 0x22222222, w & 0x44444444 and (w >> 3) & 0x11111111, whose nibbles are
//      1/2, 1, 2 and 1/2 where a bit is set.  Register d, nibble i has K position 4 i + d of the word.
//   X  in the same order, times 2, 1, 1/2 and 2 (and 1/4 in 6 bits, which the instruction's scale takes back), so
//      that every product is the code: 1 and 2 bits as 4-bit floats, 3 and 4 bits as 6-bit floats, 5 to 8 bits as two
//      of those, the upper four bits scaled by 16.  One launch makes these operands for all workgroups.
//
// A workgroup has RWV waves of 32 RT rows each below one another and 32 CT columns, and KS = 4 of such groups, which share
// the chunks of K (128 columns of A) and add up at the end through LDS.  A stage is a chunk for each group: a row's 64 bytes
// of A, which four lanes read together (lanes that read 16 bytes of 64 rows cost the cache 64 lines a load: 16384 x 16384 x
// 256 at 4 bits 57 us), and the chunks' operands of X.  Both go to LDS without passing through registers, three to six
// stages ahead, and a stage's operands from there to registers beside the products of the one in front, so that one
// barrier a stage is all the waves wait for (read in front of their own products: 57 us again).  Two waves per SIMD: one
// wave's addresses and waits are beside the other's products (one: 64 us).  Zero-tile jumping is the ascending list of the
// chunks in which a row of the workgroup has a kept tile; a stage of zeros is left out by its wave.
//
// Measured against bytes, in graphs, us: 16384 x 16384 x 256 at 4 bits 92.5 and 47.0 (of which making the operands 5, products 20
// at 6.9 POP/s, the rest the first loads, sums and output, 12, and waits for loads); at 8 bits 91.8 and 81.2; 9000 x
// 9000 x 300 at 2 bits 53.7 and 30.5; 12000 x 12000 x 100 at 8 bits 52.7 and 35.8; 8192 x 8192 x 64 at 2 bits 17.6 and 11.8.
#include "agg_dense.h"

namespace qgtc {
namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

enum { kNibbles = 0, kSixBits = 1, kTwoSixBits = 2 };      // 1 and 2 bits, 3 and 4, 5 to 8
constexpr int dense_parts(int fmt) { return fmt == kTwoSixBits ? 2 : 1; }
constexpr int dense_part_bytes(int fmt) { return fmt == kNibbles ? 512 : 768; }   // of 32 columns of a word
constexpr int dense_word_bytes(int fmt) { return dense_parts(fmt) * dense_part_bytes(fmt); }
int dense_format(int s) { return s <= 2 ? kNibbles : (s <= 4 ? kSixBits : kTwoSixBits); }

// ---- X ---------------------------------------------------------------------------------------------------
struct DenseCodes {
  const uint32_t* X;
  int64_t ld, ps;
  int32_t s, cols, kwords;
  uint8_t* dst;
  int64_t cg_bytes;          // of 32 columns
};

// Planes to operands, [32 columns][word][part][16 bytes of each column, then 8]: a thread has 32 rows of a column.
template <int FMT>
__global__ __launch_bounds__(256) void dense_codes_kernel(const DenseCodes p) {
  const unsigned idx = blockIdx.x * 256u + threadIdx.x, cg = blockIdx.y;
  const int kw = (int)(idx >> 5), c = (int)(idx & 31u);
  if (kw >= p.kwords) return;
  const uint32_t* const from = p.X + (int64_t)kw * p.ld + min((int)cg * 32 + c, p.cols - 1);
  uint32_t a[8];
#pragma unroll
  for (int pl = 0; pl < (FMT == kNibbles ? 2 : (FMT == kSixBits ? 4 : 8)); ++pl) {
    a[pl] = 0u;
    if (pl < p.s) a[pl] = from[(int64_t)pl * p.ps];
  }
  uint8_t* const to = p.dst + (int64_t)cg * p.cg_bytes + (int64_t)kw * dense_word_bytes(FMT);
  if constexpr (FMT == kNibbles) {
    v4u v;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const uint32_t b0 = (a[0] >> d) & 0x11111111u, b1 = (a[1] >> d) & 0x11111111u, b3 = b0 & b1;
      if (d == 1) v[d] = b3 | (b0 & ~b1) << 1 | b1 << 2;         // 0, 1, 2, 3
      else if (d == 2) v[d] = b0 | b1 << 1;                      // halves of these
      else v[d] = b3 | b1 << 1 | (b0 | b1) << 2;                 // doubles
    }
    *reinterpret_cast<v4u*>(to + c * 16) = v;
  } else {
#pragma unroll
    for (int part = 0; part < dense_parts(FMT); ++part) {
      uint32_t out[6];
#pragma unroll
      for (int half = 0; half < 2; ++half) {                     // registers 0 and 1, 2 and 3 of the operand of A: 16 entries, 96 bits
        uint32_t w[2][2];                                        // 24 bits each
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const int d = 2 * half + k;
          uint32_t b[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) b[i] = (a[4 * part + i] >> d) & 0x11111111u;
          // E2M3 of code / 8 (the code itself), of twice that, and of four times that: eight entries at a time
          const uint32_t m = b[3], q = m | b[2];
          uint32_t low, high;
          if (d == 2) {
            low = b[0] | b[1] << 1 | b[2] << 2 | b[3] << 3;
            high = 0u;
          } else if (d == 1) {
            low = (m & b[0]) | ((m & b[1]) | (~m & b[0])) << 1 | ((m & b[2]) | (~m & b[1])) << 2 | (~m & b[2]) << 3;
            high = m;
          } else {
            low = (m & b[0]) | ((m & b[1]) | (q & ~m & b[0])) << 1 | ((m & b[2]) | (q & ~m & b[1]) | (~q & b[0])) << 2 | (m | (~q & b[1])) << 3;
            high = q;
          }
          auto spread = [](uint32_t v) {                         // four nibbles to every sixth bit
            v = (v & 0xffu) | (v & 0xff00u) << 4;
            return (v & 0x00f00fu) | (v & 0x0f00f0u) << 2;
          };
#pragma unroll
          for (int h = 0; h < 2; ++h) w[k][h] = spread(low >> (16 * h) & 0xffffu) | spread(high >> (16 * h) & 0xffffu) << 4;
        }
        out[3 * half] = w[0][0] | w[0][1] << 24;
        out[3 * half + 1] = w[0][1] >> 8 | w[1][0] << 16;
        out[3 * half + 2] = w[1][0] >> 16 | w[1][1] << 8;
      }
      *reinterpret_cast<v4u*>(to + part * 768 + c * 16) = (v4u){out[0], out[1], out[2], out[3]};
      *reinterpret_cast<v2u*>(to + part * 768 + 512 + c * 8) = (v2u){out[4], out[5]};
    }
  }
}

// ---- the product -------------------------------------------------------------------------------------------
struct DenseParams {
  const uint32_t* A;
  const uint8_t* X;
  int64_t lda;
  int64_t cg_bytes;
  int32_t a_words;
  int32_t rows, block_rows, eff_rows;
  int32_t cols;
  int32_t n_chunks;
  int32_t n_col_wg, rb_per_sub;    // workgroups along the columns, and along the rows of a diagonal block
  uint32_t col_magic, rb_magic;
  int32_t run_shift;
  uint32_t nblocks;
  int32_t list_off;                // LDS: chunk list and mask (0: all chunks)
  int32_t n_tile_cols, tile_shift;
  const int32_t* row_cnt;
  const int32_t* col_idx;
  EpiParams ep;
};

// Whether the workgroup (its rows are tile rows tr0 .. tr0 + n_tr - 1, MOST at most) takes all chunks: a list that leaves out
// less than an eighth of them costs more than it saves (65536 x 256 columns in blocks of 4096 with 0.1 % of the bits, at 8
// bits: 138 us with such lists, 117), and one such row is enough.  Scalar loads, which need not wait for the stages that are
// on their way.
typedef const __attribute__((address_space(4))) int32_t* ScalarInts;
template <int MOST>
__device__ __forceinline__ bool dense_all_chunks(const DenseParams& p, int tr0, int n_tr) {
  const ScalarInts cnt = (ScalarInts)(uintptr_t)(p.row_cnt + (int)uniform((uint32_t)tr0));
  int most = 0;
#pragma unroll
  for (int t = 0; t < MOST; ++t) most = max(most, cnt[min(t, n_tr - 1)]);
  return most > p.n_tile_cols - p.n_tile_cols / 8 - 1;
}

// The workgroup's chunks from the tile map, and their number.
__device__ __forceinline__ int dense_list(const DenseParams& p, uint8_t* lds, int tr0, int n_tr, int n_waves) {
  uint16_t* const list = reinterpret_cast<uint16_t*>(lds + p.list_off);
  const int mw = (p.n_chunks + 31) >> 5, tid = (int)threadIdx.x, wave = tid >> 6, lane = tid & 63;
  uint32_t* const mask = reinterpret_cast<uint32_t*>(lds + p.list_off + (2 * p.n_chunks + 3) / 4 * 4);
  uint32_t* const count = mask + mw;
  for (int i = tid; i < mw; i += 64 * n_waves) mask[i] = 0u;
  __syncthreads();
  for (int t = wave; t < n_tr; t += n_waves) {
    const int cnt = p.row_cnt[tr0 + t];
    const int32_t* const idx = p.col_idx + (int64_t)(tr0 + t) * p.n_tile_cols;
    for (int i = lane; i < cnt; i += 64) {
      const int c = idx[i] >> p.tile_shift;
      atomicOr(&mask[c >> 5], 1u << (c & 31));
    }
  }
  __syncthreads();
  if (wave == 0) {
    int base = 0;
    for (int i0 = 0; i0 < mw; i0 += 64) {
      uint32_t m = i0 + lane < mw ? mask[i0 + lane] : 0u;
      if (i0 + lane == mw - 1 && (p.n_chunks & 31)) m &= (1u << (p.n_chunks & 31)) - 1u;
      int at = __builtin_popcount(m), incl = at;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
      }
      const int total = __shfl(incl, 63, 64);
      at = base + incl - at;
      while (m) {
        list[at++] = (uint16_t)(32 * (i0 + lane) + __builtin_ctz(m));
        m &= m - 1u;
      }
      base += total;
    }
    if (lane == 0) *count = (uint32_t)base;
  }
  __syncthreads();
  return (int)uniform(*count);
}

// Sums of 16 consecutive columns of row n of a tile of 32 to the output; lane ^ 32 has the row's other 16 of 32.  room: 4 KiB
// of LDS, the wave's own.
__device__ __forceinline__ void dense_emit(const DenseParams& p, int row0, int rows_here, int cg, int n, int kh, uint32_t (&y)[16],
                                           uint32_t* room) {
  const EpiParams& e = p.ep;
  const int col0 = 32 * cg + 16 * kh;
  const bool row_ok = n < rows_here;
  const int row = row0 + (row_ok ? n : 0);
  if (e.mode == QGTC_OUT_I32 || e.mode == QGTC_OUT_F32) {
    const bool vec = (e.ld_out & 3) == 0 && ((uintptr_t)e.out & 15u) == 0;   // 16-byte stores
    uint32_t* const dst = reinterpret_cast<uint32_t*>(e.out) + (int64_t)row * e.ld_out + col0;
    const double ri = e.row_i ? (double)e.row_i[row] : 0.0;
    const double l0 = e.l0a + e.l0b * (e.row_l ? (double)e.row_l[row] : 0.0);
#pragma unroll
    for (int k = 0; k < 16; k += 4) {
#pragma unroll
      for (int r = k; r < k + 4; ++r) {
        if (e.mode == QGTC_OUT_I32) {
          y[r] = (e.relu && (int32_t)y[r] < 0) ? 0u : y[r];
        } else {
          // the arithmetic of dequantize_f64, with the row terms formed once
          const int cc = min(col0 + r, p.cols - 1);
          const double t1 = e.cc * (double)(int32_t)y[r] + e.rs * ri;
          double v = t1 + l0 * (e.ck + e.cs * (e.col_i ? (double)e.col_i[cc] : 0.0));
          if (e.col_a) v = v * (double)e.col_a[cc] + (e.col_b ? (double)e.col_b[cc] : 0.0);
          if (e.relu && v < 0.0) v = 0.0;
          y[r] = __float_as_uint((float)v);
        }
      }
      if (vec && row_ok) {
        if (col0 + k + 4 <= p.cols) {
          *reinterpret_cast<v4u*>(dst + k) = (v4u){y[k], y[k + 1], y[k + 2], y[k + 3]};
        } else {
#pragma unroll
          for (int r = k; r < k + 4; ++r)
            if (col0 + r < p.cols) dst[r] = y[r];
        }
      }
    }
    // Rows that are not whole 16 bytes: through LDS, so that a store is 32 columns of two rows instead of one of 64 (8200 x 2049
    // x 257 at 8 bits, us: one by one 38.7, here 25.8; at 2 bits 29.8 and 18.6).
    if (__builtin_expect(!vec, 0)) {
#pragma unroll
      for (int k = 0; k < 16; ++k) room[32 * n + ((16 * kh + k) ^ n)] = y[k];   // (rows spread over the banks)
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      uint32_t* const to = reinterpret_cast<uint32_t*>(e.out) + (int64_t)row0 * e.ld_out + 32 * cg + n;
#pragma unroll 4
      for (int k = 0; k < 16; ++k) {
        const int r = 2 * k + kh;
        const uint32_t v = room[32 * r + (n ^ r)];
        if (r < rows_here && 32 * cg + n < p.cols) to[(int64_t)r * e.ld_out] = v;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    return;
  }
  // planes packed along the columns: 16 bits of a word per plane and lane
  const int qbits = e.rq_nbits;
  const uint32_t qmax = qbits >= 32 ? 0xffffffffu : ((1u << qbits) - 1u);
  const float qmaxf = (float)qmax;
#pragma unroll
  for (int k = 0; k < 16; ++k) y[k] = col0 + k < p.cols ? requantize_i32(y[k], min(col0 + k, p.cols - 1), e, qmax, qmaxf) : 0u;
  uint32_t* const drow = reinterpret_cast<uint32_t*>(e.out) + (int64_t)row * e.ld_out;
  for (int p0 = 0; p0 < qbits; p0 += 8) {
    uint32_t lo[2], hi[2];                           // byte i: bit p0 + i of eight codes
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      lo[b] = hi[b] = 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const uint32_t c = (y[8 * b + k] >> p0) & 0xffu;
        if (k < 4) lo[b] |= c << (8 * k);
        else hi[b] |= c << (8 * (k - 4));
      }
      transpose_bits_8x8(lo[b], hi[b]);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int sh = 8 * (i & 3);
      const uint32_t mine = (((i < 4 ? lo[0] : hi[0]) >> sh) & 0xffu) | (((i < 4 ? lo[1] : hi[1]) >> sh) & 0xffu) << 8;
      const uint32_t word = mine | (uint32_t)__shfl_xor((int)mine, 32, 64) << 16;
      if (p0 + i < qbits && row_ok && kh == 0) drow[(int64_t)(p0 + i) * e.ps_out + cg] = word;
    }
  }
  // a LEFT operand has zeros between the last data word of a row and its leading dimension
  const int data_words = (p.cols + 31) >> 5;
  if (cg == data_words - 1 && row_ok) {
    for (int pl = 0; pl < qbits; ++pl)
      for (int wd = data_words + kh; wd < (int)e.ld_out; wd += 2) drow[(int64_t)pl * e.ps_out + wd] = 0u;
  }
}

__device__ __forceinline__ v8i dense_expand(uint32_t w) {
  const int a = (int)(w & 0x11111111u), b = (int)(w & 0x22222222u), c = (int)(w & 0x44444444u), d = (int)((w >> 3) & 0x11111111u);
  return (v8i){a, b, c, d, 0, 0, 0, 0};
}
// Operand of X: column c's 16 bytes and, of six bits, 8 more; `from` is its word's and part's place.
template <int FMT>
__device__ __forceinline__ v8i dense_operand(const uint8_t* from, int c) {
  const v4i v = *reinterpret_cast<const v4i*>(from + c * 16);
  if constexpr (FMT == kNibbles) return (v8i){v.x, v.y, v.z, v.w, 0, 0, 0, 0};
  // (an address of its own: two such pieces read by one instruction would have to be moved to their operands)
  int at = 512 + c * 8;
  asm("" : "+v"(at));
  const v2u u = *reinterpret_cast<const v2u*>(from + at);
  return (v8i){v.x, v.y, v.z, v.w, (int)u.x, (int)u.y, 0, 0};
}
// scale: 2^(scale - 127)
template <int FMT, int PART>
__device__ __forceinline__ v16f dense_mfma(const v8i& x, const v8i& a, const v16f& c) {
  constexpr int SCALE = FMT == kNibbles ? 127 : (PART == 0 ? 129 : 133);
  return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(x, a, c, FMT == kNibbles ? 4 : 2, 4, 0, SCALE, 0, 127);
}

// At most `later` (up to MOST) times LOADS of the wave's loads are still on their way.
template <int LOADS, int MOST>
__device__ __forceinline__ void dense_wait(int later) {
  if constexpr (MOST > 0) {
    if (later < MOST) {
      dense_wait<LOADS, MOST - 1>(later);
      return;
    }
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0f70 | (MOST * LOADS & 15) | (MOST * LOADS >> 4) << 14);   // vmcnt
  asm volatile("" ::: "memory");
}

template <int FMT, int RT, int CT, int RWV, int KS>
struct DenseShape {
  static constexpr int WORD = dense_word_bytes(FMT), PARTS = dense_parts(FMT);
  static constexpr int ROWS = 32 * RT * RWV;         // of the workgroup
  static constexpr int X_CG = 4 * WORD;              // of 32 columns: a chunk
  static constexpr int X_PART = CT * X_CG;           // of a wave's stage
  static constexpr int NW = RWV * KS;
  static constexpr int ROW = KS * 16;                // bytes of a row of A
  static constexpr int SLOT = KS * X_PART + ROWS * ROW;
  static constexpr int MOST = 140 * 1024;            // (and up to 17 KiB of a chunk list)
  static constexpr int SLOTS = MOST / SLOT < 6 ? MOST / SLOT : 6;
  // Loads of 1 KiB that a wave issues per stage (where they do not divide evenly some are made twice).
  static constexpr int X_PIECES = X_PART / 1024, X_LOADS = (X_PIECES + RWV - 1) / RWV;
  static constexpr int A_PIECES = ROWS * ROW / 1024, A_LOADS = (A_PIECES + NW - 1) / NW;
  static constexpr int LOADS = X_LOADS + A_LOADS;
  static constexpr int TILES = RT * CT;              // 32 x 32
  static constexpr int BOX = NW * TILES * 4096;      // sums of all waves, at the end: half of the tiles at a time where there are many
  static constexpr int ROUNDS = (BOX + MOST - 1) / MOST;
  static constexpr int LDS = SLOTS * SLOT > BOX / ROUNDS ? SLOTS * SLOT : BOX / ROUNDS;
  static_assert(SLOTS >= 3 && (SLOTS - 1) * LOADS < 64 && LDS <= MOST && TILES % ROUNDS == 0 && KS == 4, "shapes");
};

template <int FMT, int RT, int CT, int RWV, int KS>
__global__ __launch_bounds__(64 * RWV * KS) void dense_kernel(const DenseParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  using Sh = DenseShape<FMT, RT, CT, RWV, KS>;
  constexpr int ROWS = Sh::ROWS;
  unsigned b = xcd_deal(blockIdx.x, p.run_shift);
  if (b >= p.nblocks) return;                        // whole workgroup leaves together
  unsigned q = div_by(b, (unsigned)p.n_col_wg, p.col_magic);
  const int cw = (int)(b - q * (unsigned)p.n_col_wg);
  b = q;
  q = div_by(b, (unsigned)p.rb_per_sub, p.rb_magic);
  const int lrow_wg = (int)(b - q * (unsigned)p.rb_per_sub) * ROWS;   // in the diagonal block q
  const int wave = (int)uniform(threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  const int rw = wave % RWV, kp = wave / RWV;
  const int n = lane & 31, kh = lane >> 5;
  // position n of the columns: a lane then has 16 sums side by side
  const int col = 16 * ((n >> 2) & 1) + 4 * (n >> 3) + (n & 3);
  const int block0 = (int)q * p.block_rows;
  const int rows_wg = min(min(p.eff_rows - lrow_wg, p.rows - block0 - lrow_wg), ROWS);
  if (rows_wg <= 0) return;                          // behind a short last block
  const int lrow = lrow_wg + rw * 32 * RT, row0 = block0 + lrow;      // the wave's first row
  const int rows_here = min(max(rows_wg - rw * 32 * RT, 0), 32 * RT);
  const int kw_base = block0 >> 5;
  const bool self = p.ep.self_term != 0;
  int n_list = p.n_chunks;
  const uint16_t* list = nullptr;

  // ---- loads of a stage ----
  const uint32_t lds0 = uniform((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds);
  const uint32_t lda4 = (uint32_t)p.lda * 4u;
  // A: 16 / KS rows of KS chunks, 16 bytes each, in a piece; the chunks of a row are in an order that spreads the rows
  // over the banks
  v4u rx[CT];
  const v4u ra = uniform_words(p.A + (uint64_t)(uint32_t)(block0 + lrow_wg) * (uint64_t)p.lda, (uint32_t)(rows_wg - 1) * lda4 + (uint32_t)p.a_words * 4u);
  const int a_chunk = (lane & (KS - 1)) ^ ((lane / KS >> 2) & (KS - 1));
#pragma unroll
  for (int k = 0; k < CT; ++k) {
    const int cg = cw * CT + k;
    rx[k] = uniform_words(p.X + (int64_t)cg * p.cg_bytes, 32 * cg < p.cols ? (uint32_t)p.cg_bytes : 0u);
  }
  const uint32_t x_lane = (uint32_t)lane * 16u, a_from = (uint32_t)(lane / KS) * lda4;
  constexpr uint32_t A_AT = KS * Sh::X_PART;
  const uint32_t x_to = (uint32_t)(kp * Sh::X_PART);
  auto load = [&](int st, uint32_t slot) {
    // (past the last chunk: A is read from behind its end, as zeros)
    const int i = st * KS + kp, ia = st * KS + a_chunk;
    int c = min(i, n_list - 1), ca = min(ia, n_list - 1);
    if (list) {
      c = (int)uniform(list[c]);
      ca = list[ca];
    }
    const uint32_t a_voff = ia < n_list ? a_from + (uint32_t)ca * 16u : 0x80000000u;
#pragma unroll
    for (int j = 0; j < Sh::A_LOADS; ++j) {
      const int piece = (j * Sh::NW + wave) % Sh::A_PIECES;
      load_lds(ra, a_voff, (uint32_t)piece * (64 / KS) * lda4, slot + A_AT + (uint32_t)piece * 1024u);
    }
#pragma unroll
    for (int j = 0; j < Sh::X_LOADS; ++j) {
      const int piece = min(j * RWV + rw, Sh::X_PIECES - 1), k = piece / (Sh::X_CG / 1024);   // of the wave's stage: column group, 1 KiB
      const uint32_t from = (uint32_t)(kw_base + 4 * c) * Sh::WORD + (uint32_t)(piece % (Sh::X_CG / 1024)) * 1024u;
      load_lds(CT == 1 || k == 0 ? rx[0] : rx[CT - 1], x_lane, from, slot + x_to + (uint32_t)piece * 1024u);
    }
  };

  // ---- products of a stage ----
  v16f acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int k = 0; k < CT; ++k)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[t][k][i] = 0.0f;
  // A lane's operands: half kh of its chunk, two words of each of its rows, and the same words of its column.
  struct Stage {
    v2u a[RT];
    v8i x[2][CT][Sh::PARTS];
  };
  const int a_at = (rw * 32 * RT + n) * Sh::ROW + ((kp ^ (n >> 2)) & (KS - 1)) * 16 + kh * 8;   // (tiles are whole turns of the order)
  auto read = [&](const uint8_t* slot, Stage& f) {
#pragma unroll
    for (int t = 0; t < RT; ++t) f.a[t] = *reinterpret_cast<const v2u*>(slot + A_AT + a_at + t * 32 * Sh::ROW);
    const uint8_t* const xs = slot + x_to + kh * 2 * Sh::WORD;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int k = 0; k < CT; ++k)
#pragma unroll
        for (int i = 0; i < Sh::PARTS; ++i) f.x[j][k][i] = dense_operand<FMT>(xs + k * Sh::X_CG + j * Sh::WORD + i * 768, col);
  };
  auto multiply = [&](const Stage& f) {
    uint32_t any = 0u;
#pragma unroll
    for (int t = 0; t < RT; ++t) any |= f.a[t].x | f.a[t].y;
    if (__builtin_amdgcn_ballot_w64(any != 0u) == 0ull) return;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const v8i e = dense_expand(f.a[t][j]);
#pragma unroll
        for (int k = 0; k < CT; ++k) {
          acc[t][k] = dense_mfma<FMT, 0>(f.x[j][k][0], e, acc[t][k]);
          if constexpr (Sh::PARTS == 2) acc[t][k] = dense_mfma<FMT, 1>(f.x[j][k][1], e, acc[t][k]);
        }
      }
  };

  // ---- the pipeline: a stage's operands go to registers beside the products of the one in front, and its slot is
  // then loaded again ----
  auto load_first = [&](int from, int upto) {
#pragma unroll 1
    for (int i = from; i < min(upto, (n_list + KS - 1) / KS); ++i) load(i, lds0 + (uint32_t)(i * Sh::SLOT));
  };
  // Of all chunks first, while the lengths of the lists come: two stages, which most lists turn out to want; more are in the way
  // of a short list's (8192 x 8192 x 64 with 8 full blocks on the diagonal, at 2 bits: all slots 9.8 us, two 9.4; 32768 x 32768
  // x 128 with blocks of 1024, at 8 bits 32.1 and 30.2).
  int from = p.list_off ? 2 : Sh::SLOTS;
  load_first(0, from);
  if (p.list_off) {
    const int tr0 = (block0 + lrow_wg) >> 4, n_tr = (rows_wg + 15) >> 4;
    if (!dense_all_chunks<ROWS / 16>(p, tr0, n_tr)) {
      n_list = dense_list(p, lds, tr0, n_tr, Sh::NW);
      list = reinterpret_cast<const uint16_t*>(lds + p.list_off);
      dense_wait<0, 0>(0);
      __syncthreads();
      from = 0;
    }
    load_first(from, Sh::SLOTS);
  }
  const int n_st = (n_list + KS - 1) / KS;
  uint32_t slot = 0;                                 // of the stage in front
  Stage fa, fb;
  auto meet = [&] {                                  // what every wave has read is in its registers
    __builtin_amdgcn_s_waitcnt(0xc07f);              // lgkmcnt(0)
    __syncthreads();
  };
  auto step = [&](Stage& now, Stage& then, int st, bool more) {
    const uint32_t at = slot;
    slot = slot == (Sh::SLOTS - 1) * Sh::SLOT ? 0u : slot + Sh::SLOT;
    if (more) dense_wait<Sh::LOADS, Sh::SLOTS - 2>(Sh::SLOTS - 2);
    else dense_wait<Sh::LOADS, Sh::SLOTS - 2>(max(n_st - 2 - st, 0));
    meet();
    read(lds + slot, then);                          // (behind the last stage: of what is there, not used)
    if (more) load(st + Sh::SLOTS, lds0 + at);
    __builtin_amdgcn_sched_barrier(0);
    multiply(now);
  };
  if (n_st > 0) {
    dense_wait<Sh::LOADS, Sh::SLOTS - 1>(min(n_st, Sh::SLOTS) - 1);
    __syncthreads();
    read(lds, fa);
  }
  int st = 0;
#pragma unroll 1
  for (; st + 1 + Sh::SLOTS < n_st; st += 2) {
    step(fa, fb, st, true);
    step(fb, fa, st + 1, true);
  }
#pragma unroll 1
  for (; st < n_st; st += 2) {
    step(fa, fb, st, st + Sh::SLOTS < n_st);
    if (st + 1 < n_st) step(fb, fa, st + 1, false);
  }
  if (self && kp == 0) {                             // the rows themselves, through an identity as A
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      if (32 * t >= rows_here) continue;
      const v8i e = dense_expand(kh == 0 ? 1u << n : 0u);
#pragma unroll
      for (int k = 0; k < CT; ++k) {
        const uint8_t* const at = p.X + (int64_t)min(cw * CT + k, (p.cols - 1) >> 5) * p.cg_bytes + (int64_t)(kw_base + (lrow >> 5) + t) * Sh::WORD;
        acc[t][k] = dense_mfma<FMT, 0>(dense_operand<FMT>(at, col), e, acc[t][k]);
        if constexpr (Sh::PARTS == 2) acc[t][k] = dense_mfma<FMT, 1>(dense_operand<FMT>(at + 768, col), e, acc[t][k]);
      }
    }
  }

  // ---- output: the groups of waves add up, and finish a share of the tiles each ----
  v4f* const box = reinterpret_cast<v4f*>(lds) + lane;
  constexpr int ROUND = Sh::TILES / Sh::ROUNDS;
#pragma unroll
  for (int r0 = 0; r0 < Sh::TILES; r0 += ROUND) {
    __syncthreads();                                 // every wave is through with what is there
#pragma unroll
    for (int i = 0; i < ROUND; ++i) {
      const v16f& v = acc[(r0 + i) / CT][(r0 + i) % CT];
#pragma unroll
      for (int k = 0; k < 4; ++k) box[((wave * ROUND + i) * 4 + k) * 64] = (v4f){v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]};
    }
    __syncthreads();
#pragma unroll 1
    for (int i = kp; i < ROUND; i += KS) {
      const int t = (r0 + i) / CT;
      int cg = cw * CT + (r0 + i) % CT;
      asm("" : "+s"(cg));                             // (the addresses of the columns' terms, out of the loop, are 80 registers)
      if (32 * cg >= p.cols || 32 * t >= rows_here) continue;
      uint32_t y[16];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        v4f v = box[((rw * ROUND + i) * 4 + k) * 64];
#pragma unroll
        for (int j = 1; j < KS; ++j) v += box[(((rw + j * RWV) * ROUND + i) * 4 + k) * 64];
#pragma unroll
        for (int r = 0; r < 4; ++r) y[4 * k + r] = (uint32_t)(int)v[r];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the sums of this tile have been read, and by this wave alone
      dense_emit(p, row0 + 32 * t, rows_here - 32 * t, cg, n, kh, y, reinterpret_cast<uint32_t*>(lds) + (rw * ROUND + i) * 1024);
    }
  }
}

template <int FMT, int RT, int CT, int RWV, int KS>
qgtc_status launch(DenseParams* dp, int xcd_run, hipStream_t stream) {
  DenseParams& p = *dp;
  using Sh = DenseShape<FMT, RT, CT, RWV, KS>;
  constexpr int ROWS = 32 * RT * RWV;
  const int n_sub = p.block_rows > 0 ? cdiv(p.rows, p.block_rows) : 1;
  p.rb_per_sub = cdiv(p.eff_rows, ROWS);
  p.n_col_wg = cdiv(p.cols, 32 * CT);
  p.rb_magic = div_magic(p.rb_per_sub);
  p.col_magic = div_magic(p.n_col_wg);
  const int64_t blocks = (int64_t)n_sub * p.rb_per_sub * p.n_col_wg;
  p.nblocks = (uint32_t)blocks;
  // a run of an XCD is whole rows of workgroups, which read the same rows of A, as far as every XCD gets one
  int64_t run = xcd_run > 0 ? (int64_t)cdiv((int64_t)xcd_run * 16, ROWS) * p.n_col_wg : cdiv(blocks, 8);
  p.run_shift = 0;
  while (((int64_t)2 << p.run_shift) <= run && p.run_shift < 24) ++p.run_shift;
  size_t lds = Sh::LDS;
  p.list_off = 0;
  if (p.row_cnt && p.n_chunks <= 8192) {
    p.list_off = (int)lds;
    lds += (size_t)((2 * p.n_chunks + 3) / 4 + cdiv(p.n_chunks, 32) + 1) * 4;
    lds = (lds + 15) & ~(size_t)15;
  }
  static OncePerDevice once;
  if (!allow_lds(once, reinterpret_cast<const void*>(&dense_kernel<FMT, RT, CT, RWV, KS>), lds)) return QGTC_ERR_HIP;
  hipLaunchKernelGGL((dense_kernel<FMT, RT, CT, RWV, KS>), dim3(xcd_deal_grid(p.nblocks, p.run_shift)), dim3(64 * Sh::NW), lds, stream, p);
  return launch_status();
}

template <int FMT, int CT>
qgtc_status launch_rows(DenseParams* p, int rows, int xcd_run, hipStream_t stream) {
  if (rows == 256) return launch<FMT, 4, CT, 2, 4>(p, xcd_run, stream);
  if (rows == 128) return launch<FMT, 2, CT, 2, 4>(p, xcd_run, stream);
  if (rows == 64) return launch<FMT, 1, CT, 2, 4>(p, xcd_run, stream);
  return launch<FMT, 1, CT, 1, 4>(p, xcd_run, stream);
}

bool one_tile(const AggParams& p) { return p.cols <= 32 || dense_format(p.s) == kTwoSixBits; }   // of columns per workgroup

// The most rows of a workgroup that give half of the compute units one: more of them read X more often, and take turns.
// 256, 128, 64 and 32 rows, us: 12000 x 12000 x 100 at 8 bits (188, 376, .. workgroups) 35.8, 44.5, 65.5, 107; 12288 x 12288 x
// 16 at 2 (48, 96, 192, ..) 21.1, 15.8, 13.3, 14.6; 8192 x 8192 x 64 at 2 (32, 64, 128, 256) 22.7, 16.1, 13.2, 11.8.
int dense_rows(const AggParams& p) {
  const int64_t half = device_compute_units() / 2;
  for (int rows = 256; rows > 32; rows >>= 1)
    if (dense_groups(p, rows) > half) return rows;
  return 32;
}

}  // namespace

// Sums, which may include the row itself, below 2^24: of 8 bits up to 65792 columns of A.
bool dense_applies(const AggParams& p) {
  return p.s <= 8 && p.lda < (int64_t)1 << 21 && (((int64_t)1 << p.s) - 1) * ((int64_t)p.a_words * 32 + 1) < (int64_t)1 << 24;
}

int64_t dense_groups(const AggParams& p, int rows) {
  const int eff = p.eff_rows < p.rows ? p.eff_rows : p.rows;
  return (int64_t)(p.block_rows > 0 ? cdiv(p.rows, p.block_rows) : 1) * cdiv(eff, rows) * cdiv(p.cols, one_tile(p) ? 32 : 64);
}

static int64_t dense_group_bytes(const AggParams& p) { return (int64_t)p.x_kwords * dense_word_bytes(dense_format(p.s)); }
int64_t dense_bytes(const AggParams& p) { return dense_group_bytes(p) * cdiv(p.cols, 32); }

qgtc_status dense_aggregate(const AggParams& a, void* workspace, int xcd_run, hipStream_t stream) {
  DenseCodes c{};
  c.X = a.X;
  c.ld = a.ldx4 / 4;
  c.ps = a.psx4 / 4;
  c.s = a.s;
  c.cols = a.cols;
  c.kwords = a.x_kwords;
  c.dst = reinterpret_cast<uint8_t*>(workspace);
  c.cg_bytes = dense_group_bytes(a);
  const int fmt = dense_format(a.s);
  const dim3 grid((unsigned)cdiv((int64_t)c.kwords * 32, 256), (unsigned)cdiv(c.cols, 32));
  if (fmt == kNibbles) hipLaunchKernelGGL(dense_codes_kernel<kNibbles>, grid, dim3(256), 0, stream, c);
  else if (fmt == kSixBits) hipLaunchKernelGGL(dense_codes_kernel<kSixBits>, grid, dim3(256), 0, stream, c);
  else hipLaunchKernelGGL(dense_codes_kernel<kTwoSixBits>, grid, dim3(256), 0, stream, c);
  const qgtc_status st = launch_status();
  if (st != QGTC_OK) return st;

  DenseParams p{};
  p.A = a.A;
  p.X = c.dst;
  p.lda = a.lda;
  p.cg_bytes = c.cg_bytes;
  p.a_words = a.a_words;
  p.rows = a.rows;
  p.block_rows = a.block_rows;
  p.eff_rows = a.eff_rows < a.rows ? a.eff_rows : a.rows;
  p.cols = a.cols;
  p.n_chunks = a.a_words / 4;
  p.n_tile_cols = a.n_tile_cols;
  p.tile_shift = a.tile_shift;
  p.row_cnt = a.row_cnt;
  p.col_idx = a.col_idx;
  p.ep = a.ep;
  const int rows = dense_rows(a);
  if (fmt == kTwoSixBits) return launch_rows<kTwoSixBits, 1>(&p, rows, xcd_run, stream);
  if (one_tile(a)) return fmt == kNibbles ? launch_rows<kNibbles, 1>(&p, rows, xcd_run, stream) : launch_rows<kSixBits, 1>(&p, rows, xcd_run, stream);
  return fmt == kNibbles ? launch_rows<kNibbles, 2>(&p, rows, xcd_run, stream) : launch_rows<kSixBits, 2>(&p, rows, xcd_run, stream);
}

}  // namespace qgtc
