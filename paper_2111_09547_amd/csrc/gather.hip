// Host side of the fused layer over neighbour lists (gather_kernel.h), and features in its form
// from packed planes.
#include "gather.h"

namespace qgtc {
namespace {

struct PlanesParams {
  const uint32_t* X;
  int64_t ld, ps;
  int32_t rows, cols, s;
  uint8_t* dst;
  int32_t ld_dst;            // bytes
  uint32_t flip;
  int32_t parts;             // 2: planes from 8 on behind the others, in the second half of a row
};

// Planes to bytes: a thread has 32 rows of four columns, whose plane words it transposes as 8 x 8 bit
// matrices; eight rows at a time its bytes are put in row order and stored as words.
__global__ __launch_bounds__(256) void planes_to_rows_kernel(const PlanesParams p) {
  const int part = (int)blockIdx.y, quads = p.ld_dst / p.parts / 4;
  const unsigned idx = blockIdx.x * 256u + threadIdx.x;
  const int kw = (int)(idx / (unsigned)quads), c0 = 4 * (int)(idx % (unsigned)quads);
  if (kw * 32 >= p.rows) return;
  uint32_t code[4][8];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int c = min(c0 + k, p.cols - 1);
#pragma unroll
    for (int pl = 0; pl < 8; ++pl) {
      code[k][pl] = 0u;
      if (8 * part + pl < p.s) code[k][pl] = p.X[(int64_t)(8 * part + pl) * p.ps + (int64_t)kw * p.ld + c];
    }
    planes_word_to_codes(code[k]);
    if (c0 + k >= p.cols) {
#pragma unroll
      for (int r = 0; r < 8; ++r) code[k][r] = 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    // byte b of the four words: row 8 b + r
    const uint32_t lo01 = __builtin_amdgcn_perm(code[1][r], code[0][r], 0x05010400u), hi01 = __builtin_amdgcn_perm(code[1][r], code[0][r], 0x07030602u);
    const uint32_t lo23 = __builtin_amdgcn_perm(code[3][r], code[2][r], 0x05010400u), hi23 = __builtin_amdgcn_perm(code[3][r], code[2][r], 0x07030602u);
    const uint32_t v[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                           __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int row = 32 * kw + 8 * b + r;
      if (row < p.rows) *reinterpret_cast<uint32_t*>(p.dst + (int64_t)row * p.ld_dst + 4 * quads * part + c0) = v[b] ^ p.flip;
    }
  }
}

}  // namespace

qgtc_status planes_to_rows(const qgtc_bits* X, uint8_t* dst, hipStream_t stream) {
  const int parts = X->nbits > 8 ? 2 : 1, ld = (int)row_codes_ld(X->cols);
  PlanesParams p{X->data, X->ld_words, X->plane_stride_words, X->rows, X->cols, X->nbits, dst, parts * ld,
                 parts == 2 ? 0x80808080u : row_codes_flip(X->nbits), parts};
  ProfScope prof(QGTC_KERNEL_PACK, stream);
  hipLaunchKernelGGL(planes_to_rows_kernel, dim3((unsigned)cdiv((int64_t)cdiv(p.rows, 32) * (ld / 4), 256), (unsigned)parts), dim3(256), 0,
                     stream, p);
  return launch_status();
}

void gather_weights(GatherParams* p, const qgtc_bits* W) {
  p->wb = reinterpret_cast<const uint8_t*>(W->data);
  p->wb_part = W->plane_stride_words * 4;
  p->h = W->cols;
  p->n_nt = cdiv(W->cols, 16);
  p->n_ks = cdiv(W->rows, 64);
  p->split_y = p->agg_nbits == 8;
  p->split_w = W->nbits == 8;
  p->sum_parts = 1;
}

namespace {

// A tile per wave where that gives every compute unit eight waves (65536 rows, 64 -> 64: 8.8 us, with four waves
// per tile 11.3; 8192 rows have half a wave per SIMD that way).
bool four_waves_share(const GatherParams& p) { return p.ldx > 32 && p.n_tiles < 8 * device_compute_units(); }

int pieces_of(const GatherParams& p, int parts = 1) {
  int pieces = 1;
  while (16 * pieces * parts < p.ldx) pieces <<= 1;
  return pieces;
}
size_t heavy_bytes(const GatherParams& p, int parts = 1) { return 2048 + 64 + (size_t)pieces_of(p, parts) * 64 * parts; }   // counts, the row that is taken, its sums

void set_grid(GatherParams* gp, int tiles) {
  GatherParams& p = *gp;
  const int cus = device_compute_units();
  p.nblocks = (uint32_t)cdiv(p.n_tiles, tiles);
  // workgroups that read the same rows of X stay on one XCD, as far as every XCD still gets a run
  int64_t run = cdiv(cdiv(p.block, 16), tiles);
  if (run > (int64_t)p.nblocks / 8) run = p.nblocks / 8;
  p.run_shift = 0;
  while (((int64_t)2 << p.run_shift) <= run && p.run_shift < 24) ++p.run_shift;
  // Two per compute unit.  A visit for nothing costs the tiles more than half a microsecond per 512 of them (65536 rows, 16 -> 16 ->
  // 16, without heavy rows: 20.1 us, with 1024 of them 20.9), and rows of more columns take as long as the caches deliver them
  // (with 512 and 1024, us: 64 -> 64 -> 64 on 262144 rows of a power-law graph 80.0 and 82.9, 524288 130 and 133; 48 columns
  // 66.8 and 69.6, 32 59.0 and 61.4; 512 -> 16 on 262144 75 and 82).  Of 16 columns, whose rows are round trips and
  // little else, four from 262144 rows on: sums of 16 at 4 bits, twice, behind 512 -> 16 127.9 and 121.4, 16 -> 16 -> 16 47.1 and
  // 44.4 (1540 heavy rows; with smaller blocks and fewer of them 39.3 and 40.8, without any 36.5 and 37.1).
  const int most = (p.ldx <= 16 && p.n_groups >= 16 * cus ? 4 : 2) * cus;
  p.n_heavy_wg = p.block > kListLight ? (p.n_groups < most ? (p.n_groups + 7) / 8 * 8 : most / 8 * 8) : 0;
}

}  // namespace

qgtc_status gather_layer(GatherParams* gp, int mode, const qgtc_bits* W, hipStream_t stream) {
  GatherParams& p = *gp;
  gather_weights(gp, W);
  if (p.up.l0b == 0.0) p.up.row_l = nullptr;
  p.want_rowsum = p.up.mode == QGTC_OUT_F32 && p.up.row_i == nullptr && p.up.rs != 0.0;
  const bool share = four_waves_share(p);
  const int tiles = share ? 1 : 4;
  const int n_ntp = share || p.n_nt == 1 ? p.n_nt : (p.n_nt + 3) / 4 * 4;
  // The codes of a tile: of 256 columns at a time where one group of output tiles is all.  Heavy rows,
  // one at a time, need those of all columns.
  const bool parts = pieces_of(p) > 16 && !share && p.n_nt <= (p.n_nt == 1 ? 1 : 4);
  size_t lds = (size_t)tiles * (parts ? 4 : p.n_ks) * 1024;
  const size_t one = (size_t)p.n_ks * 1024;
  p.heavy_off = (int)one;
  if (lds < one + heavy_bytes(p)) lds = one + heavy_bytes(p);
  lds = (lds + 63) & ~(size_t)63;
  p.cols_off = (int)lds;
  lds += (size_t)n_ntp * (64 + 128);
  p.w_off = -1;
  if (p.n_ks * n_ntp <= 48) {
    p.w_off = (int)lds;
    lds += (size_t)p.n_ks * n_ntp * 1024;
  }
  set_grid(gp, tiles);
  ProfScope prof(QGTC_KERNEL_LAYER, stream);
  switch (mode) {
    case kGatherCodes: return gather_launch<kGatherCodes, 1>(p, share, lds, stream);
    case kGatherAffine: return gather_launch<kGatherAffine, 1>(p, share, lds, stream);
    default: return gather_launch<kGatherRows, 1>(p, share, lds, stream);
  }
}

qgtc_status gather_wide_layer(GatherParams* gp, int mode, const qgtc_bits* low, const qgtc_bits* high, hipStream_t stream) {
  GatherParams& p = *gp;
  gather_weights(gp, low);
  p.split_y = 1;                                     // (kept_codes(): every byte minus 128)
  p.wb_high = high ? reinterpret_cast<const uint8_t*>(high->data) : nullptr;
  p.w_parts = high ? 2 : 1;
  p.split_w_high = high && high->nbits == 8;
  p.sum_parts = 2;
  if (p.up.l0b == 0.0) p.up.row_l = nullptr;
  p.want_rowsum = p.up.mode == QGTC_OUT_F32 && p.up.row_i == nullptr && p.up.rs != 0.0;
  const bool share = p.ldx > 64 && p.n_tiles < 8 * device_compute_units();
  const int tiles = share ? 1 : 4;
  size_t lds = (size_t)tiles * 2 * p.n_ks * 1024;
  const size_t one = (size_t)2 * p.n_ks * 1024;
  p.heavy_off = (int)one;
  if (lds < one + heavy_bytes(p, 2)) lds = one + heavy_bytes(p, 2);
  lds = (lds + 63) & ~(size_t)63;
  p.cols_off = (int)lds;
  lds += (size_t)p.n_nt * (128 + 128);
  p.w_off = -1;
  if (p.n_ks * p.n_nt * p.w_parts <= 48) {
    p.w_off = (int)lds;
    lds += (size_t)p.n_ks * p.n_nt * p.w_parts * 1024;
  }
  set_grid(gp, tiles);
  ProfScope prof(QGTC_KERNEL_LAYER, stream);
  switch (mode) {
    case kGatherCodes: return gather_launch<kGatherCodes, 2>(p, share, lds, stream);
    case kGatherAffine: return gather_launch<kGatherAffine, 2>(p, share, lds, stream);
    default: return gather_launch<kGatherRows, 2>(p, share, lds, stream);
  }
}

qgtc_status gather_sums(GatherParams* gp, hipStream_t stream) {
  const bool share = four_waves_share(*gp);
  set_grid(gp, share ? 1 : 4);
  ProfScope prof(QGTC_KERNEL_AGGREGATE, stream);
  return gather_launch<kGatherSums, 1>(*gp, share, heavy_bytes(*gp), stream);
}

}  // namespace qgtc
