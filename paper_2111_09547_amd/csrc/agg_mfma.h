// The aggregation on the int8 matrix cores, shared by the stand-alone kernel
// (aggregate.hip) and by the fused layer kernel (layer_kernel.h).
//
// A is binary, X has up to 8 planes per pass: Y = A.X is the integer product of 0/1 bytes
// with the codes of X, so one v_mfma_i32_16x16x64_i8 takes 16 rows x 16 columns x 64 K
// positions of ALL planes at once.  What is left to do is to bring both operands into bytes:
//   A  one adjacency word w becomes eight operand registers (w >> b) & 0x01010101, b = 0..7
//      (a word per lane is 16 rows by 128 K positions: 15 vector instructions, ~36 cycles, and
//      2 CT matrix instructions of 16); register b holds K positions b, b + 8, b + 16, b + 24.
//   X  the eight plane words of 32 rows of a column are transposed as 8 x 8 bit matrices
//      (planes_word_to_codes): code word r holds rows r, r + 8, r + 16, r + 24 - the same
//      order.  This is done once per workgroup while X is staged into LDS; between the
//      layers of a stack X is kept in this form (layer.h) and staging it is a copy.
// The instruction is signed: codes of 8 planes enter as code - 128 (one XOR per word), and
// 128 x (bits of the row of A) is added back at the end.
//
// Work split.  A unit is 64 rows of A (four 16-row tiles).  WAYS waves share it, each with its
// own 16 CT columns and all of K, so that no sums are exchanged; a workgroup has up to four
// units side by side that read the same staged rows of X.  G = 16 CT WAYS columns are done at a
// time; more columns are further passes over the same rows.  Where rows are few and long, KS
// waves take each column part, every one its share of each stage, and add up at the end.
//   operand M = columns of X: position m of tile ft of a group of 16 LT columns is column
//     4 LT (m / 4) + 4 ft + m % 4; a wave takes CT tiles of a group, so that a lane ends up with
//     4 CT consecutive columns of one node
//   operand N = nodes: position n of tile t is row 32 (t / 2) + 8 (n % 4) + 4 (t % 2) + n / 4 of
//     the unit.  A result of the update (nodes along M, see layer_kernel.h) then has the nodes
//     4 (t % 2) + g + {0, 8, 16, 24} of a word row in one lane: the four bytes of one code word
//     of the next X.
// K is taken in chunks of 128 (four words of A, four word rows of X), SWC chunks per stage.
// Which chunks: all of them, or (zero-tile jumping, Section 4.3 of the paper) the ascending
// list of those in which one of the workgroup's rows has a kept tile.  A stage whose words are
// zero in all 64 rows of a unit is left out by its waves (one ballot).
//   lane group g = lane / 16 takes words SWC g .. SWC g + SWC - 1 of the stage's 4 SWC words.
//
// Pipeline.  X in operand order and the words of A go to LDS without passing through registers
// (4 to 16 KiB of X and SWC KiB of A per unit and stage), two stages ahead, through three slots with
// one barrier per stage; the matrix cores' time per stage is 256 to 512 cycles per wave.
// What bounds it is a stage's latency and its barrier: 16384 x 16384 x 256 at 4 bits, 96 us, is two waves per SIMD, whose
// vector instructions take 38 us and matrix instructions 31, and which wait a third of their time; 8192 x 8192 x 64 at 2 bits,
// 18 us, 6.4 and 2 us, and half of the time.
#pragma once
#include <type_traits>

#include "qgtc_internal.h"

namespace qgtc {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

constexpr int kUnitRows = 64;
constexpr int kMaxUnits = 4;

enum { kSrcPlanes = 0, kSrcCodes = 1 };

// Sizes of a split; lt: 16-column tiles per column group of the staged order.
struct AggSplit {
  int ct, ways, lt, ks;
  constexpr int group() const { return 16 * ct * ways; }
  constexpr int wave_chunks() const { return group() == 128 ? 1 : 2; }   // per stage
  constexpr int chunks() const { return wave_chunks() * ks; }
  constexpr int x_bytes() const { return chunks() * 128 * group(); }                      // staged X
  constexpr int slot_bytes(int nu) const { return x_bytes() + nu * chunks() * 1024; }
};
constexpr int kSlots = 3;

struct AggParams {
  const uint32_t* A;
  const uint32_t* X;       // planes (RIGHT) or codes (kSrcCodes, see codes_offset())
  int64_t lda;             // words per row of A
  int32_t a_words;         // readable words per row (data rounded up to 128 bits)
  int32_t rows;            // rows of A (= output rows)
  int32_t block_rows;      // 0, or rows per diagonal block
  int32_t eff_rows;        // rows of a diagonal block (of the whole matrix without blocks)
  uint32_t x_bytes;        // bytes spanned by X (codes: by one column group)
  uint32_t ldx4, psx4;     // planes: bytes between word rows / planes of X
  int32_t x_kwords;        // word rows of X
  int32_t s;               // planes of X
  int32_t cols;            // columns of X (= output columns)
  // launch shape
  int32_t n_chunks;        // 128-wide chunks of K that a row of A can touch
  int32_t n_col_wg;        // workgroups along the columns
  int32_t n_pass;          // passes of G columns
  int32_t nu, n_waves;     // units side by side, waves (WAYS KS nu)
  int32_t sub_per_wg;      // diagonal blocks a workgroup covers (> 1 only for blocks of at most 128 rows)
  int32_t ups_log2;        // log2 of the units per block where sub_per_wg > 1
  int32_t rb_per_sub;      // workgroups per diagonal block
  uint32_t rb_magic, col_magic;   // div_magic() of rb_per_sub and n_col_wg
  int32_t slot_bytes;      // one LDS slot
  int32_t list_off;        // LDS offset (bytes) of the chunk list (0: all chunks), behind it the chunk mask
  int32_t run_shift;       // log2 of the run of consecutive workgroups one XCD takes
  uint32_t nblocks;
  int32_t n_tile_rows, n_tile_cols;
  int32_t tile_shift;      // log2 of tiles per chunk
  const int32_t* row_cnt;  // tile map (NULL: all tiles)
  const int32_t* col_idx;
  EpiParams ep;
};

// Checks the adjacency of an aggregation and its map, and fills their part of the kernel parameters.
inline qgtc_status agg_fill_adjacency(const qgtc_bits* A, const qgtc_tile_map* map, AggParams* p) {
  qgtc_status st = check_adjacency(A);
  if (st != QGTC_OK) return st;
  if (A->ld_words * 64 >= (int64_t)1 << 31) return QGTC_ERR_UNSUPPORTED;
  p->A = A->data;
  p->lda = A->ld_words;
  p->a_words = 4 * cdiv(A->cols, 128);
  p->rows = A->rows;
  p->block_rows = A->block_rows;
  p->eff_rows = A->block_rows > 0 ? A->block_rows : A->rows;
  if (map) {
    if (!map->row_cnt || !map->col_idx) return QGTC_ERR_NULL;
    if (map->tile_rows != 16 ||
        (map->tile_kbits != 32 && map->tile_kbits != 64 && map->tile_kbits != 128))
      return QGTC_ERR_UNSUPPORTED;
    if (map->n_tile_rows != cdiv(A->rows, 16) || map->n_tile_cols != cdiv(A->cols, map->tile_kbits))
      return QGTC_ERR_SHAPE;
    p->row_cnt = map->row_cnt;
    p->col_idx = map->col_idx;
    p->n_tile_rows = map->n_tile_rows;
    p->n_tile_cols = map->n_tile_cols;
    p->tile_shift = map->tile_kbits == 128 ? 0 : (map->tile_kbits == 64 ? 1 : 2);
  }
  return QGTC_OK;
}

// Checks the operands of an aggregation and fills the operand part of the kernel
// parameters (everything but the epilogue and the launch shape).
inline qgtc_status agg_fill_params(const qgtc_bits* A, const qgtc_tile_map* map, const qgtc_bits* X,
                                   AggParams* p) {
  if (!A || !X) return QGTC_ERR_NULL;
  qgtc_status st = check_adjacency(A);
  if (st != QGTC_OK) return st;
  st = check_bits(X, QGTC_RIGHT);
  if (st != QGTC_OK) return st;
  if (A->block_rows > 0) {
    if (A->rows != X->rows) return QGTC_ERR_SHAPE;
  } else if (A->cols != X->rows) {
    return QGTC_ERR_SHAPE;
  }
  const int64_t x_words = span_words(X);
  if (x_words * 4 >= (int64_t)1 << 32 || X->ld_words * 4 >= (int64_t)1 << 31 ||
      X->plane_stride_words * 4 >= (int64_t)1 << 31)
    return QGTC_ERR_UNSUPPORTED;
  p->X = X->data;
  p->ldx4 = (uint32_t)(X->ld_words * 4);
  p->psx4 = (uint32_t)(X->plane_stride_words * 4);
  p->x_bytes = (uint32_t)(x_words * 4);
  p->x_kwords = cdiv(X->rows, 32);
  p->s = X->nbits;
  p->cols = X->cols;
  return agg_fill_adjacency(A, map, p);
}

// n / d by the upper half of n * div_magic(d), for any n below 2^31: the rounded-up reciprocal is
// too large by less than 1 / 2^32, so the product by less than one, and the quotient is at most
// one too large.  (A runtime division costs ~30 instructions, and the code in front of the first
// load is fetched cold by every launch.)
inline uint32_t div_magic(int d) { return d <= 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + (uint64_t)d - 1) / (uint64_t)d); }
__host__ __device__ __forceinline__ unsigned div_by(unsigned n, unsigned d, uint32_t magic) {
  const unsigned q = magic ? (unsigned)(((uint64_t)n * magic) >> 32) : n;
  return q - (unsigned)(q * d > n);
}

// A wave addresses its rows of A with 32 bits: 64 rows where one wave has a unit, 32 or fewer where
// several share it, which rows of 64 MiB and more need.
inline bool agg_long_rows(int64_t lda) { return lda >= (int64_t)1 << 24; }

// The split of a stand-alone aggregation of `cols` columns.
AggSplit aggregate_split(int rows, int cols, int a_words, int64_t lda);

// A tile map is worth its loads (two dependent ones in front of the first stage) where the list of
// chunks can save stages: for rows of more than 1024 columns with diagonal blocks, of more than one
// stage without.
inline bool agg_reads_map(const AggParams& p, const AggSplit& sp) {
  return p.sub_per_wg == 1 && p.n_chunks <= 8192 && p.n_chunks > (p.block_rows > 0 ? 8 : sp.chunks());
}

// Launch shape for a split; n_col_wg: workgroups along the columns.
// Returns the dynamic LDS that the aggregation needs.
//   Units side by side: as many (at most four, and eight waves) as leave every compute unit a
//   workgroup: they share one staged copy of X.
inline size_t agg_set_shape(AggParams* p, const AggSplit& sp, int n_col_wg, int xcd_run) {
  const int cus = device_compute_units();
  const int n_sub = p->block_rows > 0 ? cdiv(p->rows, p->block_rows) : 1;
  const int ups = cdiv(p->eff_rows, kUnitRows);
  p->n_col_wg = n_col_wg;
  p->n_pass = cdiv(p->cols, sp.group() * n_col_wg);
  p->n_chunks = p->a_words / 4;
  const int64_t units = (int64_t)n_sub * ups * n_col_wg;
  const int upw = sp.ways * sp.ks;                   // waves per unit
  int nu = upw == 4 ? 2 : kMaxUnits;
  while (nu > 1 && units < (int64_t)nu * cus) nu >>= 1;
  if (nu * upw < 2) nu = 2;
  p->sub_per_wg = 1;
  p->ups_log2 = ups > 1 ? 1 : 0;
  if (p->block_rows > 0 && p->block_rows <= 128 && nu / ups > 1) {
    // the staged word rows begin with the first block's
    p->sub_per_wg = 4 * sp.chunks() / (p->block_rows / 32);
    if (p->sub_per_wg > nu / ups) p->sub_per_wg = nu / ups;
    if (p->sub_per_wg < 1) p->sub_per_wg = 1;
  }
  if (p->sub_per_wg > 1) {
    p->rb_per_sub = 1;
    nu = p->sub_per_wg * ups;
  } else {
    p->rb_per_sub = cdiv(ups, nu);
    nu = cdiv(ups, p->rb_per_sub);
    if (nu * upw < 2) nu = 2;
  }
  p->nu = nu;
  p->n_waves = nu * upw;
  p->rb_magic = div_magic(p->rb_per_sub);
  p->col_magic = div_magic(n_col_wg);
  const int64_t n_rb = p->sub_per_wg > 1 ? cdiv(n_sub, p->sub_per_wg) : (int64_t)n_sub * p->rb_per_sub;
  p->nblocks = (uint32_t)(n_rb * n_col_wg);
  // Workgroups that read the same rows of X stay on one XCD (and its L2), as far as every
  // XCD still gets a run.
  int64_t run = p->rb_per_sub;
  if (run > (int64_t)p->nblocks / 8) run = p->nblocks / 8;
  if (xcd_run > 0) run = cdiv((int64_t)xcd_run * 16, (int64_t)nu * kUnitRows);
  if (xcd_run < 0) run = cdiv(p->nblocks, 8);
  int sh = 0;
  while (((int64_t)2 << sh) <= run && sh < 24) ++sh;
  p->run_shift = sh;
  p->slot_bytes = sp.slot_bytes(nu);
  size_t lds = (size_t)p->slot_bytes * kSlots;
  p->list_off = 0;
  if (p->row_cnt && agg_reads_map(*p, sp)) {
    p->list_off = (int)lds;
    lds += (size_t)((2 * p->n_chunks + 3) / 4 + cdiv(p->n_chunks, 32) + 1) * 4;
    lds = (lds + 15) & ~(size_t)15;
  }
  return lds;
}

// Place of column c of a group in the staged order (see the top): tile, position m.
template <int LT>
__device__ __forceinline__ int staged_pos(int c) {
  return 16 * ((c >> 2) % LT) + 4 * (c / (4 * LT)) + (c & 3);
}
// First of the 4 CT columns of lane group g of a wave, within the pass.
template <int CT, int LT>
__device__ __forceinline__ int lane_columns(int way, int g) {
  return way * CT / LT * (16 * LT) + 4 * LT * g + way * CT % LT * 4;
}

// A wave-uniform value in a scalar register (the compiler computes some of them lane by lane;
// a buffer descriptor that is not scalar is read through a loop over the lanes' values).
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ __amdgpu_buffer_rsrc_t uniform_rsrc(const void* base, uint32_t bytes) {
  const uint64_t b = (uint64_t)base;
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)uniform((uint32_t)(b >> 32)) << 32) | uniform((uint32_t)b)), 0,
                                           (int)uniform(bytes), 0x00020000);
}

// What a wave is in its workgroup.
struct AggWave {
  int wave, u, way, kp;  // wave, unit, column part, part of the stages
  int cw;                // workgroup along the columns
  int row0, rows_here;   // first row of the unit, rows it has (<= 0: none)
  int kw_base;           // first word row of X of the workgroup's chunk 0
  int klds;              // word rows between the workgroup's and the unit's first word row
  int own_kw;            // word of A that holds the unit's first 32 rows (self term)
  int n_list;            // chunks to take
};

// Rows of unit w->u of workgroup b (host and device).
__host__ __device__ __forceinline__ void agg_locate(const AggParams& p, unsigned b, AggWave* w) {
  unsigned q = div_by(b, (unsigned)p.rb_per_sub, p.rb_magic);
  const int j = (int)(b - q * (unsigned)p.rb_per_sub);
  b = q;
  q = div_by(b, (unsigned)p.n_col_wg, p.col_magic);
  w->cw = (int)(b - q * (unsigned)p.n_col_wg);
  const int bw = p.block_rows >> 5;
  int sub = (int)q * p.sub_per_wg, lrow = (j * p.nu + w->u) * kUnitRows;
  w->kw_base = sub * bw;
  w->klds = 0;
  if (p.sub_per_wg > 1) {
    const int sl = w->u >> p.ups_log2;
    sub += sl;
    lrow = (w->u & ((1 << p.ups_log2) - 1)) * kUnitRows;
    w->klds = sl * bw;
  }
  w->row0 = sub * p.block_rows + lrow;
  w->own_kw = lrow >> 5;
  const int in_block = p.eff_rows - lrow, in_all = p.rows - w->row0;
  const int here = in_block < in_all ? in_block : in_all;
  w->rows_here = here < kUnitRows ? here : kUnitRows;
}

// False: no work for this workgroup (it leaves as a whole).
template <int WAYS, int KS>
__device__ __forceinline__ bool agg_place(const AggParams& p, AggWave* w) {
  const unsigned b = xcd_deal(blockIdx.x, p.run_shift);
  if (b >= p.nblocks) return false;
  w->wave = (int)uniform(threadIdx.x >> 6);
  w->u = w->wave / (WAYS * KS);
  w->way = w->wave % WAYS;
  w->kp = w->wave / WAYS % KS;
  agg_locate(p, b, w);
  w->n_list = p.n_chunks;
  return true;
}

// The list of the workgroup's chunks from the tile map (LDS; ends with a barrier).
template <int WAYS, int KS>
__device__ __forceinline__ void agg_list(const AggParams& p, AggWave* w, uint8_t* lds, bool self_term) {
  if (p.list_off == 0) return;                       // uniform
  uint16_t* list = reinterpret_cast<uint16_t*>(lds + p.list_off);
  const int mw = (p.n_chunks + 31) >> 5;
  uint32_t* mask = reinterpret_cast<uint32_t*>(lds + p.list_off + (2 * p.n_chunks + 3) / 4 * 4);
  uint32_t* count = mask + mw;
  // the waves of a unit share its four tile rows; the first 64 entries of a list are requested
  // beside its length
  constexpr int TR = 4 / (WAYS * KS), PARTS = WAYS * KS;
  const int lane = threadIdx.x & 63;
  const int part = w->wave % PARTS;
  const int tr0 = (w->row0 >> 4) + TR * part;
  int cnt[TR], first[TR];
#pragma unroll
  for (int t = 0; t < TR; ++t) {
    cnt[t] = first[t] = 0;
    if (w->rows_here > 16 * (TR * part + t)) {
      cnt[t] = p.row_cnt[tr0 + t];
      first[t] = p.col_idx[(int64_t)(tr0 + t) * p.n_tile_cols + min(lane, p.n_tile_cols - 1)];
    }
  }
  for (int i = threadIdx.x; i < mw; i += p.n_waves * 64) mask[i] = 0u;
  __syncthreads();
  bool all = false;
#pragma unroll
  for (int t = 0; t < TR; ++t) {
    if (cnt[t] >= p.n_tile_cols) {                   // a full list is not read
      all = true;
      continue;
    }
    const int32_t* rest = p.col_idx + (int64_t)(tr0 + t) * p.n_tile_cols;
    for (int i = lane; i < cnt[t]; i += 64) {
      const int c = (i < 64 ? first[t] : rest[i]) >> p.tile_shift;
      atomicOr(&mask[c >> 5], 1u << (c & 31));
    }
  }
  if (self_term && w->rows_here > 0 && lane == 0) {
    const int c = w->own_kw >> 2;
    atomicOr(&mask[c >> 5], 1u << (c & 31));
  }
  if (all)
    for (int i = lane; i < mw; i += 64) atomicOr(&mask[i], 0xffffffffu);
  __syncthreads();
  if (w->wave == 0) {
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
    if (lane == 0) {
      if (base == 0) list[0] = 0;                    // (one chunk of zeros keeps the loops simple)
      *count = base == 0 ? 1u : (uint32_t)base;
    }
  }
  __syncthreads();
  w->n_list = (int)uniform(*count);
}

// Wave-wide loads of 16 bytes per lane straight to LDS address `to` (+ 16 lane).  Written as
// assembly because the compiler, which sees such a load as a store to LDS, would make every
// later read of LDS wait for it: nothing would overlap.  wait_loads() and a barrier complete them.
// The scalar offset is held to the buffer's size: the unit compares the lane's offset with size -
// scalar offset, which must not wrap (a unit without rows has size 0, stages past the last chunk
// lie behind the end).
__device__ __forceinline__ void load_lds(const v4u& rsrc, uint32_t voff, uint32_t soff, uint32_t to) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :: "v"(voff), "s"(rsrc), "s"(min(soff, rsrc.z)), "s"(to) : "memory", "m0");
}
__device__ __forceinline__ void load_lds_2k(const v4u& rsrc, uint32_t voff, uint32_t soff, uint32_t to) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds\n\t"
               "buffer_load_dwordx4 %0, %1, %2 offen offset:1024 lds"
               :: "v"(voff), "s"(rsrc), "s"(min(soff, rsrc.z)), "s"(to) : "memory", "m0");
}
// At most about n of the wave's loads are still on their way.
__device__ __forceinline__ void wait_loads(int n) {
  asm volatile("" ::: "memory");
  if (n >= 9) __builtin_amdgcn_s_waitcnt(0x0f79);
  else if (n >= 5) __builtin_amdgcn_s_waitcnt(0x0f75);
  else if (n >= 3) __builtin_amdgcn_s_waitcnt(0x0f73);
  else if (n >= 1) __builtin_amdgcn_s_waitcnt(0x0f71);
  else __builtin_amdgcn_s_waitcnt(0x0f70);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ v4u uniform_words(const void* base, uint32_t bytes) {
  const uint64_t b = (uint64_t)base;
  return (v4u){uniform((uint32_t)b), uniform((uint32_t)(b >> 32)), uniform(bytes), 0x00020000u};
}

// All passes over the workgroup's rows, planes plane0 .. plane0 + 7.  After each one
//   finish(pass, acc, deg)
// is called by every wave with acc = A . (codes, minus 128 when there are eight planes) of the
// wave's columns and deg = 128 x bits per row of A (0 without the offset):
//   acc[t][ft][r] of lane (n = lane % 16, g) is node n of tile t, column lane_columns() + 4 ft + r.
// `before` is run in front of the first loads, `beside` while they are on their way; what it
// writes to LDS is visible from the first finish on.
template <int CT, int WAYS, int LT, int KS, int SRC, int NPT, class Before, class Beside, class Finish>
__device__ __forceinline__ void agg_run(const AggParams& p, const AggWave& w, uint8_t* lds, int plane0, bool self_term,
                                        Before before, Beside beside, Finish finish) {
  constexpr AggSplit SP{CT, WAYS, LT, KS};
  constexpr int SWC = SP.wave_chunks(), TSC = SP.chunks();   // chunks of a stage: of a wave, of all
  constexpr int G = SP.group();
  constexpr int KB = 512 * LT;                       // bytes of a staged word row of a column group
  constexpr int GROUP_BYTES = 4 * TSC * KB;
  constexpr int X_BYTES = SP.x_bytes();
  constexpr int RPW = kUnitRows / WAYS;              // rows of A that a wave loads
  constexpr int A_WAVE = SWC * RPW * 16;             // bytes of them per stage
  constexpr int AI = (SWC * RPW + 63) / 64;          // loads of them per stage
  constexpr int PAIRS = TSC * WAYS * CT;             // 2 KiB pieces of X per stage: TSC LT of each group
  const int tid = (int)threadIdx.x;
  const int lane = tid & 63;
  const int ln = lane & 15, g = lane >> 4;
  const int np = min(p.s - plane0, 8);
  const bool offset = np == 8;
  // (a list of all chunks is the same without it)
  const uint16_t* list = p.list_off && w.n_list != p.n_chunks ? reinterpret_cast<const uint16_t*>(lds + p.list_off) : nullptr;
  const int n_st = (w.n_list + TSC - 1) / TSC;
  const int x_last = p.sub_per_wg > 1 ? TSC - 1 : w.n_list - 1;
  const int c_wave = w.kp * SWC;                     // the wave's first chunk of a stage
  const int cg_wg = w.cw * p.n_pass * (G / (16 * LT));   // first column group of the workgroup
  const uint32_t lds0 = uniform((uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds);

  // ---- loads of a stage ----
  const uint32_t lda4 = (uint32_t)p.lda * 4u;
  const int a_rows = min(w.rows_here - w.way * RPW, RPW);   // the wave's
  const v4u ra = uniform_words(p.A + (uint64_t)(uint32_t)(w.row0 + w.way * RPW) * (uint64_t)p.lda,
                               a_rows > 0 ? (uint32_t)(a_rows - 1) * lda4 + (uint32_t)p.a_words * 4u : 0u);
  // (the stage is a scalar offset where all chunks are taken)
  const uint32_t arow = (uint32_t)(lane % RPW) * lda4, a_chunk = (uint32_t)(lane / RPW);
  const uint32_t a_to = (uint32_t)(X_BYTES + w.u * TSC * 1024 + w.kp * SWC * 1024 + w.way * A_WAVE);
  auto load_a = [&](int st, uint32_t slot) {
#pragma unroll
    for (int k = 0; k < AI; ++k) {
      const uint32_t c = a_chunk + (uint32_t)(k * (64 / RPW));   // chunk of the stage
      uint32_t voff = arow + c * 16u, soff = (uint32_t)(st * TSC + c_wave) * 16u;
      if (list) {                                    // uniform
        voff = arow + (uint32_t)list[min(st * TSC + c_wave + (int)c, w.n_list - 1)] * 16u;
        soff = 0u;
      }
      // (chunks past the last one are read from the next rows, or as zeros, and not used)
      if (SWC * RPW >= 64 || lane < SWC * RPW) load_lds(ra, voff, soff, slot + a_to + (uint32_t)(k * 1024));
    }
  };
  // 2 KiB piece q of a stage of X: TSC LT pieces of each column group
  const uint32_t x_lane = (uint32_t)lane * 16u;
  auto x_rsrc = [&](int pass, int q) {
    const int cg = cg_wg + pass * (G / (16 * LT)) + q / (TSC * LT);
    const uint64_t base = (uint64_t)p.X + (uint64_t)(uint32_t)cg * p.x_bytes;
    return (v4u){(uint32_t)base, (uint32_t)(base >> 32), cg * 16 * LT < p.cols ? p.x_bytes : 0u, 0x00020000u};
  };
  auto x_from = [&](int q, int ch) { return (uint32_t)(w.kw_base + 4 * ch) * KB + (uint32_t)(q % LT * 2048); };
  auto x_to = [&](int q) { return (uint32_t)(q / (TSC * LT) * GROUP_BYTES + q / LT % TSC * 4 * KB + q % LT * 2048); };
  // (the usual case: all chunks in order and at most one piece per wave and stage)
  const bool one_piece = !list && p.n_waves >= PAIRS;
  const uint32_t from0 = x_from(w.wave, w.wave / LT % TSC), to0 = x_to(w.wave);
  v4u rx0 = x_rsrc(0, w.wave);
  int rx0_pass = 0;
  auto load_x_codes = [&](int pass, int st, uint32_t slot) {
    if (one_piece) {
      if (PAIRS < 8 && w.wave >= PAIRS) return;
      if (pass != rx0_pass) {
        rx0 = x_rsrc(pass, w.wave);
        rx0_pass = pass;
      }
      load_lds_2k(rx0, x_lane, from0 + (uint32_t)(st * (TSC * 4 * KB)), slot + to0);
      return;
    }
    for (int q = w.wave; q < PAIRS; q += p.n_waves) {
      const int ci = min(st * TSC + q / LT % TSC, x_last);
      load_lds_2k(x_rsrc(pass, q), x_lane, x_from(q, list ? (int)uniform(list[ci]) : ci), slot + x_to(q));
    }
  };
  const int x_loads = w.wave < PAIRS ? 2 * ((PAIRS - 1 - w.wave) / p.n_waves + 1) : 0;
  // planes: item i of the stage is column i % G of word row i / G
  uint32_t raw[SRC == kSrcCodes ? 1 : NPT][8];
  auto load_x_planes = [&](int pass, int st) {
    const __amdgpu_buffer_rsrc_t rx = uniform_rsrc(p.X, p.x_bytes);
    const uint32_t col4 = (uint32_t)min(cg_wg * 16 * LT + pass * G + tid % G, p.cols - 1) * 4u;
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      const int kl = tid / G + k * (p.n_waves * 64 / G);
      const int ci = min(st * TSC + (kl >> 2), x_last);
      const int ch = list ? (int)list[ci] : ci;
      const int kw = min(w.kw_base + 4 * ch + (kl & 3), p.x_kwords - 1);
      const uint32_t voff = (uint32_t)kw * p.ldx4 + col4;
#pragma unroll
      for (int pl = 0; pl < 8; ++pl) {
        raw[k][pl] = 0u;
        if (pl < np) raw[k][pl] = __builtin_amdgcn_raw_buffer_load_b32(rx, voff, (uint32_t)(plane0 + pl) * p.psx4, 0);
      }
    }
  };
  auto store_x_planes = [&](uint8_t* slot) {
    const int c = tid % G;
    uint8_t* const to = slot + c / (16 * LT) * GROUP_BYTES + staged_pos<LT>(c % (16 * LT)) * 16;
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
      const int kl = tid / G + k * (p.n_waves * 64 / G);
      planes_word_to_codes(raw[k]);
      if (offset) {
#pragma unroll
        for (int r = 0; r < 8; ++r) raw[k][r] ^= 0x80808080u;
      }
      // Every wave has its planes here, also one without a piece to store: they were requested
      // after the stage's words of A, and loads complete in order, so that these have arrived
      // as well before the wave goes to the next barrier.
#pragma unroll
      for (int r = 0; r < 8; ++r) asm volatile("" : "+v"(raw[k][r]));
      if (kl < 4 * TSC) {
        *reinterpret_cast<v4u*>(to + kl * KB) = (v4u){raw[k][0], raw[k][1], raw[k][2], raw[k][3]};
        *reinterpret_cast<v4u*>(to + kl * KB + LT * 256) = (v4u){raw[k][4], raw[k][5], raw[k][6], raw[k][7]};
      }
    }
  };

  // ---- products of a stage ----
  v4i acc[4][CT];
  uint32_t deg[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int ft = 0; ft < CT; ++ft) acc[t][ft] = (v4i){0, 0, 0, 0};
  // 64 rows x 16 CT columns x (one word of each of the four lane groups): two halves of 64 K positions
  auto read_x = [&](const uint8_t* b, v4i (&x)[2][CT]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int ft = 0; ft < CT; ++ft) x[h][ft] = *reinterpret_cast<const v4i*>(b + h * LT * 256 + ft * 256);
  };
  auto step = [&](const v4i (&x)[2][CT], const uint32_t (&wd)[4]) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        v4i e;
#pragma unroll
        for (int r = 0; r < 4; ++r) e[r] = (int)((wd[t] >> (4 * h + r)) & 0x01010101u);
#pragma unroll
        for (int ft = 0; ft < CT; ++ft) acc[t][ft] = __builtin_amdgcn_mfma_i32_16x16x64_i8(x[h][ft], e, acc[t][ft], 0, 0, 0);
      }
  };
  // this lane's words of A in a slot (tile 0): row 8 (n % 4) + n / 4, words SWC g ..
  const int r0 = 8 * (ln & 3) + (ln >> 2);
  const uint32_t a_at = (uint32_t)(X_BYTES + w.u * TSC * 1024 + w.kp * SWC * 1024 + r0 / RPW * A_WAVE +
                                   ((SWC * g >> 2) * RPW + r0 % RPW) * 16 + (SWC * g & 3) * 4);
  const uint32_t x_at = (uint32_t)(w.way * CT / LT * GROUP_BYTES + (w.klds + 4 * c_wave + SWC * g) * KB + (w.way * CT % LT * 16 + ln) * 16);
  int own_q = self_term ? w.own_kw >> 2 : -1;        // place of the unit's own chunk in the list
  if (self_term && list) {
    const uint32_t* mask = reinterpret_cast<const uint32_t*>(lds + p.list_off + (2 * p.n_chunks + 3) / 4 * 4);
    const int c = own_q;
    int below = 0;
    for (int i = 0; i < (c >> 5); ++i) below += __builtin_popcount(mask[i]);
    below += __builtin_popcount(mask[c >> 5] & ((1u << (c & 31)) - 1u));
    own_q = (int)uniform((uint32_t)below);
  }
  auto products = [&](const uint8_t* slot, int st, bool count) {
    uint32_t aw[4][SWC];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint8_t* from = slot + a_at + (t & 1) * 64 + (t >> 1) * (RPW == 64 ? 512 : SWC * 512);
      static_assert(SWC == 1 || SWC == 2, "words of A a lane reads at once");
      if constexpr (SWC == 2) {
        const v2u v = *reinterpret_cast<const v2u*>(from);
        aw[t][0] = v.x;
        aw[t][SWC - 1] = v.y;
      } else {
        aw[t][0] = *reinterpret_cast<const uint32_t*>(from);
      }
    }
    const int left = w.n_list - st * TSC - c_wave;   // the wave's chunks of the stage that exist
    if (TSC > 1 && left < SWC) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < SWC; ++i) aw[t][i] = (SWC * g >> 2) < left ? aw[t][i] : 0u;
    }
    const uint8_t* b = slot + x_at;
    v4i x[SWC][2][CT];
#pragma unroll
    for (int i = 0; i < SWC; ++i) read_x(b + i * KB, x[i]);
    uint32_t any = 0u;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int i = 0; i < SWC; ++i) any |= aw[t][i];
    if (__builtin_amdgcn_ballot_w64(any != 0u) != 0ull) {
#pragma unroll
      for (int i = 0; i < SWC; ++i) {
        const uint32_t wd[4] = {aw[0][i], aw[1][i], aw[2][i], aw[3][i]};
        step(x[i], wd);
      }
      // the next operand of A is formed between the products of this one
      __builtin_amdgcn_sched_group_barrier(2, 8, 0);
#pragma unroll
      for (int i = 0; i < SWC * 8 * CT; ++i) {
        __builtin_amdgcn_sched_group_barrier(8, 1, 0);
        __builtin_amdgcn_sched_group_barrier(2, 8 / CT, 0);
      }
    }
    if (count) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < SWC; ++i) deg[t] += __builtin_popcount(aw[t][i]);
    }
    const int own_c = own_q - st * TSC - c_wave;
    if (own_q >= 0 && own_c >= 0 && own_c < SWC) {
      // GIN self term: the unit's own rows once more, through identity blocks of A
      const int f = 4 * own_c + (w.own_kw & 3) - SWC * g;   // the own word among the lane's
      const uint32_t bit = 1u << r0;
#pragma unroll
      for (int i = 0; i < SWC; ++i) {
        const uint32_t b0 = f == i ? bit : 0u, b1 = f + 1 == i ? bit : 0u;
        const uint32_t id[4] = {b0, b0 << 4, b1, b1 << 4};
        step(x[i], id);
        if (count) {
#pragma unroll
          for (int t = 0; t < 4; ++t) deg[t] += id[t] != 0u ? 1u : 0u;
        }
      }
    }
  };
  auto end_pass = [&](int pass) {
    if (offset && pass == 0) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        deg[t] += (uint32_t)__shfl_xor((int)deg[t], 16, 64);
        deg[t] += (uint32_t)__shfl_xor((int)deg[t], 32, 64);
        deg[t] <<= 7;
      }
    }
    finish(pass, acc, deg);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int ft = 0; ft < CT; ++ft) acc[t][ft] = (v4i){0, 0, 0, 0};
  };

  // ---- the pipeline; stage (pass, st) is the it-th of `total` ----
  const int total = p.n_pass * n_st;
  const uint32_t lds_end = lds0 + (uint32_t)(kSlots * p.slot_bytes);
  int l_pass = 0, l_st = 0;                          // the stage to load next
  uint32_t l_at = lds0;
  auto load_next = [&]() {                           // (of planes: the words of A)
    if constexpr (SRC == kSrcCodes) load_x_codes(l_pass, l_st, l_at);
    load_a(l_st, l_at);
    l_at += (uint32_t)p.slot_bytes;
    if (l_at == lds_end) l_at = lds0;
    if (++l_st == n_st) {
      l_st = 0;
      ++l_pass;
    }
  };
  int pass = 0, st = 0, slot = 0;
  if constexpr (SRC == kSrcCodes) {
    before();
    load_next();
    if (total > 1) load_next();
    beside();
    for (int it = 0; it < total; ++it) {
      wait_loads(it + 1 < total ? x_loads + AI : 0);
      __syncthreads();
      if (it + 2 < total) load_next();
      products(lds + slot * p.slot_bytes, st, offset && pass == 0);
      if (++slot == kSlots) slot = 0;
      if (++st == n_st) {
        end_pass(pass);
        st = 0;
        ++pass;
      }
    }
  } else {
    // A two stages ahead; X one stage ahead in LDS - its planes are put together behind the
    // products of the stage before, while other waves are still at theirs - and two in registers.
    // (the planes of a stage are requested after its words of A: with them, those have arrived -
    // store_x_planes() sees to it that every wave waits for its planes)
    before();
    int x_pass = 0, x_st = 0;
    auto planes_next = [&]() {
      load_x_planes(x_pass, x_st);
      if (++x_st == n_st) {
        x_st = 0;
        ++x_pass;
      }
    };
    load_next();
    planes_next();
    if (total > 1) load_next();
    beside();
    store_x_planes(lds);
    if (total > 1) planes_next();
    for (int it = 0; it < total; ++it) {
      __syncthreads();
      if (it + 2 < total) load_next();
      products(lds + slot * p.slot_bytes, st, offset && pass == 0);
      if (++slot == kSlots) slot = 0;
      if (it + 1 < total) {
        store_x_planes(lds + slot * p.slot_bytes);
        if (it + 2 < total) planes_next();
      }
      if (++st == n_st) {
        end_pass(pass);
        st = 0;
        ++pass;
      }
    }
  }
}

// 16-column tiles per column group of codes (see codes_offset()) for `cols` columns.
inline int agg_col_tiles(int cols) { return cols <= 16 ? 1 : (cols <= 32 ? 2 : 4); }

// Items of a stage of planes per thread.
inline int agg_items_per_thread(const AggParams& p, const AggSplit& sp) {
  const int n = cdiv(4 * sp.chunks() * sp.group(), 64 * p.n_waves);
  return n <= 1 ? 1 : (n <= 2 ? 2 : 4);
}

}  // namespace qgtc
