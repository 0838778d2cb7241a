// One quantized GNN layer over neighbour lists (lists.h): the fused layer of layer_kernel.h for
// graphs of a few neighbours per node, where the products of whole tiles of A are mostly with zeros.
//
// X is kept as bytes, row-major, so that a neighbour is one piece of memory of up to 1 KiB:
//   1. Aggregation.  A load brings 16 columns (a piece) of four neighbours of each of 16 slots, a slot
//      being a row of A and one of its P = 2^LP pieces: lane (n, g) has neighbour 4 k + g of slot n.
//      The matrix cores add them up: with the operand A[m][16 g + b] = (b == m),
//      v_mfma_i32_16x16x64_i8 adds byte m of the four lanes of a slot to sum m of it, so that a load of
//      64 x 16 bytes costs one instruction instead of some 50 of the vector ALUs (which halves a
//      layer's instructions), and sums are exact in 32 bits.  Lists end in kListNone, which lies past
//      the end of X: such a load gives zeros and costs no traffic.
//      Heavy rows are left out, and taken one by one by workgroups of their own: from their list, or
//      from the words of A where that does not hold all neighbours.
//   2. Requantization: lane (n, g) has columns 4 g .. 4 g + 3 of slot n.  The codes of a tile of 16
//      rows go to LDS, [64 columns][row][64 bytes].
//   3. Update and epilogue as in layer_kernel.h, weights along M.  Codes are stored 16 bytes per lane:
//      the weights of 64 columns are dealt to four tiles so that a lane has 16 columns side by side.
// WPT = 1: a wave has a tile, and waits for nobody but the weights.  WPT = 4: four waves share a tile, where
// there are few.  LT: 16-column output tiles at a time.
// What bounds it at every width: latency, of four dependent loads behind a launch of 2.4 us and, in wide rows, of the
// 4 KiB that a wave has in flight.  Waves wait 57 to 71 % of their time; the vector ALUs' 320 to 450 instructions per
// wave are a third of the time of 64 -> 64 on 65536 rows, and 512 -> 16 reads at 2.1 TB/s.  Whole tiles and lists, us:
// 65536 rows in blocks of 1024, 9 neighbours, 64 -> 64 13.2 and 9.0, 128 -> 128 19.5 and 15.0; 8192 rows,
// 64 -> 64 8.6 and 4.1; 262144 rows of a power-law graph, 512 -> 16 159 and 72 (134 MB of codes: 27 at the
// rate of a copy), 1024 -> 64 on 65536 rows 168 and 95; without heavy rows 512 -> 16 320 and 64.
// Waves in flight decide in wide rows: 512 -> 16 has five per SIMD (95 registers); with four and three it took 9 and 23 us longer.
// Adding bytes up on the vector ALUs instead: 64 -> 64 11.0 us.  Heavy rows in the tiles' own waves: 512 -> 16
// on the power-law graph 232 us.
#pragma once
#include "gather_shape.h"
#include "gather_update.h"

namespace qgtc {
namespace {

// At the end of a loop that is left right behind its last product: the compiler (ROCm 7.2) copies the
// sums at the loop's head two wait states after it, where the instruction needs seven, and the copy is
// then of the old values.
__device__ __forceinline__ void settle(v4i& sum) { asm volatile("s_nop 7" : "+v"(sum)); }

// A[m][16 g + b] = (b == m), which adds up the bytes of the four lanes of a slot.
__device__ __forceinline__ v4i adder(int ln) {
  const uint32_t mark = 1u << (8 * (ln & 3));
  return (v4i){(int)((ln >> 2) == 0 ? mark : 0u), (int)((ln >> 2) == 1 ? mark : 0u),
               (int)((ln >> 2) == 2 ? mark : 0u), (int)((ln >> 2) == 3 ? mark : 0u)};
}
__device__ __forceinline__ uint32_t list_entry(const v2u& idx, int k) { return k & 1 ? idx[k >> 1] >> 16 : idx[k >> 1] & 0xffffu; }

// Keeps the compiler from moving loads behind products that could wait for them, for fewer registers than a wave may
// have.  us with and without: 64 -> 64 on 65536 rows 8.8 and 9.6, fp32 out 12.4 and 12.9; 300 columns on 15221 rows,
// 14 neighbours, 22.6 and 24.8 (all 16 entries at once), but 512 -> 16 on 262144 rows of a power-law graph 13 us more (four waves per SIMD).
template <bool ON>
__device__ __forceinline__ void all_in_flight() {
  if constexpr (ON) __builtin_amdgcn_sched_barrier(0);
}

// Rows of X that a row of A can have as neighbours: its diagonal block's.
struct Neighbours {
  __amdgpu_buffer_rsrc_t rx;
  uint32_t ldx, part;                                // bytes of a row, of a part of it
  __device__ __forceinline__ Neighbours(const GatherParams& p, int row0, int parts) {
    const int first_row = (int)div_by((unsigned)row0, (unsigned)p.block, p.block_magic) * p.block;
    ldx = (uint32_t)p.ldx;
    part = ldx / (uint32_t)parts;
    rx = uniform_rsrc(p.X + (int64_t)first_row * p.ldx, (uint32_t)(min(p.rows - first_row, p.block) * p.ldx));
  }
  __device__ __forceinline__ v4i load(uint32_t idx, uint32_t pofs) const {
    return (v4i)__builtin_amdgcn_raw_buffer_load_b128(rx, __umul24(idx, ldx) + pofs, 0, 0);
  }
  // past the end where a row has no such piece
  __device__ __forceinline__ uint32_t piece_offset(int piece) const { return 16u * (uint32_t)piece < part ? 16u * (uint32_t)piece : 0x80000000u; }
};

// Sums of four columns from col on as the output (kGatherSums).
__device__ __forceinline__ void emit_sums(const GatherParams& p, int row, int col, const v4i& sum) {
  const EpiParams& u = p.up;
  uint32_t res[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (u.mode == QGTC_OUT_I32) res[r] = (uint32_t)(u.relu ? max(sum[r], 0) : sum[r]);
    else res[r] = __float_as_uint(dequantize_f64((uint32_t)sum[r], row, min(col + r, p.cols - 1), u));
  }
  uint32_t* const dst = reinterpret_cast<uint32_t*>(u.out) + (int64_t)row * u.ld_out + col;
  if (col + 4 <= p.cols) {
    *reinterpret_cast<v4u_a4*>(dst) = (v4u){res[0], res[1], res[2], res[3]};
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (col + r < p.cols) dst[r] = res[r];
  }
}

// The heavy rows, one after the other, by all n_heavy_wg workgroups.  A chain of round trips per row, three rows per workgroup
// in the largest graphs: which row, its degree, its list or words, the codes.  A row is found by a wave's lanes at once and
// words are taken up to eight at a time, us with both one by one and here: 512-16-16 on 262144 rows of a power-law graph
// (1540 heavy rows, 236 of them from words) 199.9 and 196.4, update first 131.0 and 126.9, 128-32-32-16 on 131072 72.8 and 69.4
// (without heavy rows 172, 110 and 54).
// From 65 columns on the loads of a row's step are kept in front of its products: the compiler otherwise gives them one or
// two registers in turn, a round trip per product.  On power-law graphs, us without and with: 454 -> 64 on 8192 rows 50.8
// and 30.3, 700 -> 64 51.3 and 37.3, 200 -> 64 26.2 and 21.1, 128 -> 128 -> 64 29.6 and 26.9.  Narrower rows have several in a step
// anyway, and more registers cost their tiles a wave (16 -> 16 -> 16 on 262144 rows 44.4 and 46.1).
template <int LP, int LT, int MODE, int PARTS>
__device__ __forceinline__ void heavy_rows(const GatherParams& p, uint8_t* lds, int wave, int lane) {
  using Sh = GatherShape<LP, 1, PARTS>;
  constexpr int P = Sh::P, PS = Sh::PS, RC = Sh::RC, HV = Sh::HV;
  const int ln = lane & 15, g = lane >> 4;
  const int self = p.self_term, ldx = p.ldx, n_ks = p.n_ks;
  // their number in front of each thread's groups
  uint32_t* const before = reinterpret_cast<uint32_t*>(lds + p.heavy_off);   // [256], then [256] of the thread's own
  int32_t* const taken = reinterpret_cast<int32_t*>(lds + p.heavy_off + 2048);
  uint32_t* const sums = reinterpret_cast<uint32_t*>(lds + p.heavy_off + 2048 + 64);
  const int per = (p.n_groups + 4095) / 4096 * 16;   // groups of a thread
  uint32_t mine = 0u;
  for (int i = 0; i < per; i += 16) {
    const int at = (int)threadIdx.x * per + i;
    v4u v = {0u, 0u, 0u, 0u};
    if (at < p.n_groups) v = *reinterpret_cast<const v4u*>(p.heavy_cnt + at);   // (whole pieces)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int left = p.n_groups - at - 4 * c;    // counts that exist
      const uint32_t m = (uint32_t)((1ull << (8 * min(max(left, 0), 4))) - 1ull);
      mine = __builtin_amdgcn_sad_u8(v[c] & m, 0u, mine);
    }
  }
  uint32_t incl = mine;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t up = (uint32_t)__shfl_up((int)incl, d, 64);
    if (lane >= d) incl += up;
  }
  if (lane == 63) taken[4 + wave] = (int32_t)incl;
  __syncthreads();
  uint32_t base = 0u, all = 0u;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t c = (uint32_t)taken[4 + w];
    if (w < wave) base += c;
    all += c;
  }
  if (blockIdx.x >= all) return;                   // whole workgroup
  before[threadIdx.x] = base + incl - mine;
  before[256 + threadIdx.x] = mine;
  if constexpr (PARTS == 2) stage_wide_weights<MODE>(p, lds, wave, lane);
  else if constexpr (MODE != kGatherSums) stage_weights<LT, MODE>(p, lds, wave, lane);
  uint8_t* const yb = lds;
  const uint32_t flip = p.split_y ? 0x80808080u : 0u;
  if (MODE != kGatherSums && P < 4 && (lane & 3) >= P) {   // columns no lane has
    for (int i = 0; i < PARTS; ++i) *reinterpret_cast<v4u*>(yb + i * n_ks * 1024 + lane * 16) = (v4u){flip, flip, flip, flip};
  }
  const v4i ident = adder(ln), zero = {0, 0, 0, 0};
  const Rq q = make_rq(p.agg_lo, p.agg_relu, p.agg_inv, p.agg_nbits);
#pragma unroll 1
  for (uint32_t tile = blockIdx.x; tile < all; tile += (uint32_t)p.n_heavy_wg) {
    __syncthreads();                                 // what the last row left has been read
    // Heavy row number `tile`: the thread whose groups have it, then the group, by all of a wave's lanes at once.
    if (wave == 0) {
      int at = 0;
      uint32_t left = 0u;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t k = tile - before[64 * i + lane];
        const unsigned long long has = __builtin_amdgcn_ballot_w64(tile >= before[64 * i + lane] && k < before[256 + 64 * i + lane]);
        if (has) {
          const int l = __builtin_ctzll(has);
          at = (64 * i + l) * per;
          left = (uint32_t)__builtin_amdgcn_readlane((int)k, l);
        }
      }
      for (;; at += 64) {                            // (`per` counts hold it)
        const uint32_t c = at + lane < p.n_groups ? p.heavy_cnt[at + lane] : 0u;
        uint32_t upto = c;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t up = (uint32_t)__shfl_up((int)upto, d, 64);
          if (lane >= d) upto += up;
        }
        const unsigned long long past = __builtin_amdgcn_ballot_w64(upto > left);
        if (past || at + 64 >= p.n_groups) {
          const int l = past ? __builtin_ctzll(past) : 63;
          left -= (uint32_t)__builtin_amdgcn_readlane((int)(upto - c), l);
          at = min(at + l, p.n_groups - 1);
          break;
        }
        left -= (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
      }
      uint64_t m = p.heavy[at];
      for (; left > 0u; --left) m &= m - 1u;
      if (lane == 0) taken[0] = min(at * kListGroup + (m ? __builtin_ctzll(m) : 0), p.rows - 1);
    }
    for (int i = (int)threadIdx.x; i < P * 16 * PARTS; i += 256) sums[i] = 0u;
    __syncthreads();
    const int row0 = (int)uniform((uint32_t)taken[0]);
    const Neighbours nb(p, row0, PARTS);
    int32_t rl = 0;
    if (MODE == kGatherRows && p.up.mode == QGTC_OUT_F32 && p.up.row_l) rl = p.up.row_l[row0];
    // the waves and the slots of a unit share the row's neighbours; the sums of its columns meet in LDS
    const int n = (int)uniform((uint32_t)p.deg[row0]);
    const int rs = ln / PS;
#pragma unroll 1
    for (int hv = 0; hv < HV * PARTS; ++hv) {
      const int piece = (ln & (PS - 1)) + 16 * (hv % HV), part = hv / HV;
      const uint32_t pofs = nb.piece_offset(piece) + (uint32_t)part * nb.part;
      v4i h = zero;
      if (n <= kListMax) {
#pragma unroll 1
        for (int e = (wave * RC + rs) * kListBlock; __builtin_amdgcn_ballot_w64(e < n) != 0ull; e += 4 * RC * kListBlock) {
          v2u idx = {~0u, ~0u};
          if (e < n) idx = *reinterpret_cast<const v2u*>((e == 0 ? p.first + (int64_t)row0 * kListBlock : p.rest + (int64_t)row0 * p.rest_cap + (e - kListBlock)) + 4 * g);
          v4i y[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) y[k] = nb.load(list_entry(idx, k), pofs);
          all_in_flight<RC <= 2>();
#pragma unroll
          for (int k = 0; k < 4; ++k) h = mfma_i8(ident, y[k], h);
          settle(h);
        }
      } else {
        const uint32_t* words = p.A + (int64_t)row0 * p.lda;
#pragma unroll 1
        for (int k0 = 0; k0 < p.a_words; k0 += 256) {
          uint32_t word = 0u;
          if (k0 + 4 * lane + wave < p.a_words) word = words[k0 + 4 * lane + wave];
          unsigned long long some = __builtin_amdgcn_ballot_w64(word != 0u);
#pragma unroll 1
          while (some) {
            // several words at a time: a word's loads are up to eight, and a round trip
            constexpr int STEPS = RC < 8 ? 8 / RC : 1, NB = 8 / STEPS;
            v4i y[NB * STEPS];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
              const int l = some ? __builtin_ctzll(some) : 0;
              const uint32_t wd = some ? (uint32_t)__builtin_amdgcn_readlane((int)word, l) : 0u;
              some &= some - 1ull;
              const uint32_t col = (uint32_t)(k0 + 4 * l + wave) * 32u;
#pragma unroll
              for (int s = 0; s < STEPS; ++s) {
                const uint32_t bit = (uint32_t)((s * RC + rs) * 4 + g);
                y[b * STEPS + s] = nb.load(bit < 32u && ((wd >> (bit & 31u)) & 1u) ? col + bit : (uint32_t)kListNone, pofs);
              }
            }
            all_in_flight<RC <= 2>();
#pragma unroll
            for (int s = 0; s < NB * STEPS; ++s) h = mfma_i8(ident, y[s], h);
            settle(h);
          }
        }
      }
      if (wave == 0) {                             // (once: the own row, and 128 for every code that is code - 128)
        uint32_t own = 0u;
        if (self && 16u * (uint32_t)piece < nb.part) own = *reinterpret_cast<const uint32_t*>(p.X + (int64_t)row0 * ldx + pofs + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (rs == 0) h[r] += p.x_offset * (n + self) + (int)(int8_t)(own >> (8 * r));
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) atomicAdd(&sums[16 * P * part + 16 * piece + 4 * g + r], (uint32_t)h[r]);
    }
    __syncthreads();
    if constexpr (MODE == kGatherSums) {
      for (int i = (int)threadIdx.x; 4 * i < p.cols; i += 256)
        emit_sums(p, row0, 4 * i, (v4i){(int)sums[4 * i], (int)sums[4 * i + 1], (int)sums[4 * i + 2], (int)sums[4 * i + 3]});
      continue;
    }
    for (int i = (int)threadIdx.x; i < 4 * P && i < 16 * n_ks; i += 256) {   // four columns each
      uint8_t* const to = yb + (i >> 4) * 1024 + (i & 15) * 4;
      uint32_t c[1][4];
#pragma unroll
      for (int r = 0; r < 4; ++r) c[0][r] = sums[4 * i + r] + (PARTS == 2 ? sums[16 * P + 4 * i + r] << 8 : 0u);
      if constexpr (PARTS == 2) {
        uint32_t lo, hi;
        wide_codes(p, c[0], lo, hi);
        *reinterpret_cast<uint32_t*>(to) = kept_codes(p, lo, 4 * i);
        *reinterpret_cast<uint32_t*>(to + n_ks * 1024) = kept_codes(p, hi, 4 * i);
      } else {
        uint32_t d[1];
        pack_codes_words(c, q, d);
        *reinterpret_cast<uint32_t*>(to) = kept_codes(p, d[0], 4 * i);
      }
    }
    __syncthreads();
    if constexpr (PARTS == 2) finish_wide_tile<MODE>(p, lds, yb, row0, ln == 0, wave, 4, rl, lane);
    else finish_tile<LT, MODE>(p, lds, yb, row0, ln == 0, LT * wave, 4 * LT, rl, lane);
  }
}

template <int LP, int WPT, int LT, int MODE, int PARTS, int WAVES>
__global__ __launch_bounds__(256, WAVES) void gather_layer_kernel(const GatherParams p) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  using Sh = GatherShape<LP, WPT, PARTS>;
  constexpr int P = Sh::P, PS = Sh::PS, RC = Sh::RC, HV = Sh::HV, UNITS = Sh::UNITS, W = Sh::W;
  static_assert(WPT == 1 || (WPT == 4 && P >= 4 && LT == 1), "shapes");
  const int wave = (int)uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (__builtin_expect((int)blockIdx.x < p.n_heavy_wg, 0)) {
    heavy_rows<LP, LT, MODE, PARTS>(p, lds, wave, lane);
    return;
  }
  const unsigned b = xcd_deal(blockIdx.x - (unsigned)p.n_heavy_wg, p.run_shift);
  if (b >= p.nblocks) return;                        // whole workgroup leaves together
  const int ln = lane & 15, g = lane >> 4;
  const int tile = WPT == 1 ? (int)b * 4 + wave : (int)b;
  const int row0 = tile * 16, n_rows = min(p.rows - row0, 16);   // (none for a wave behind the last tile)
  const int self = p.self_term, ldx = p.ldx, n_ks = p.n_ks;

  // ---- lists: lane (row n of the tile, g) has the first block's entries g, 4 + g, 8 + g, 12 + g --------
  // What lies past the last row reads as zeros: sums of column 0, which nobody stores.
  const uint32_t here = (uint32_t)max(n_rows, 0);
  const __amdgpu_buffer_rsrc_t r_first = uniform_rsrc(p.first + (int64_t)row0 * kListBlock, here * (kListBlock * 2)),
                               r_deg = uniform_rsrc(p.deg + row0, here * 4);
  const v2u t_idx = __builtin_amdgcn_raw_buffer_load_b64(r_first, ln * (kListBlock * 2) + 8 * g, 0, 0);
  int t_n = (int)__builtin_amdgcn_raw_buffer_load_b32(r_deg, ln * 4, 0, 0);
  int32_t rl = 0;
  if (MODE == kGatherRows && p.up.mode == QGTC_OUT_F32 && p.up.row_l && ln < n_rows) rl = p.up.row_l[row0 + ln];
  if constexpr (PARTS == 2) stage_wide_weights<MODE>(p, lds, wave, lane);
  else if constexpr (MODE != kGatherSums) stage_weights<LT, MODE>(p, lds, wave, lane);
  const bool out_ok = ln < n_rows && t_n <= kListLight;
  if (t_n > kListLight) t_n = -1;                    // (heavy: what comes out is not stored, the row is written by others)
  const uint32_t flip = p.split_y ? 0x80808080u : 0u;
  // one group of output tiles: the codes of 256 columns at a time
  const bool parts = HV > 1 && WPT == 1 && PARTS == 1 && p.n_nt <= LT;
  uint8_t* const yb = lds + (WPT == 1 ? wave * (parts ? 4 : PARTS * n_ks) * 1024 : 0);   // the tile's codes
  if (MODE != kGatherSums && P < 4 && (lane & 3) >= P) {   // columns no lane has
    for (int i = 0; i < PARTS; ++i) *reinterpret_cast<v4u*>(yb + i * n_ks * 1024 + lane * 16) = (v4u){flip, flip, flip, flip};
  }
  if (WPT == 1 && MODE != kGatherSums) {             // waits for the weights here, and for nobody later
    __syncthreads();
  }
  if (WPT == 1 && n_rows <= 0) return;

  // ---- 1, 2: the tile's codes ---------------------------------------------------------------------
  const v4i ident = adder(ln);
  const Rq q = make_rq(p.agg_lo, p.agg_relu, p.agg_inv, p.agg_nbits);
  const Neighbours nb(p, row0, PARTS);
  const uint32_t own_size = here * (uint32_t)ldx;
  const __amdgpu_buffer_rsrc_t r_own = uniform_rsrc(p.X + (int64_t)row0 * ldx, own_size);
  constexpr int LR = Sh::LR;
  const uint32_t v_own = own_lane_offset<Sh>(ln, g, (uint32_t)ldx);
  const int first_row = WPT == 1 ? 0 : wave * (16 / WPT);   // of the wave in the tile
  const bool row_sums = p.split_w || (MODE == kGatherRows && p.want_rowsum);
  v4i z[LT], rs = {0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < LT; ++j) z[j] = rs;
#pragma unroll 1
  for (int hv = 0; hv < HV; ++hv) {
    const int piece = (ln & (PS - 1)) + 16 * hv;
    if (HV > 1 && 256 * hv >= p.cols) break;         // (uniform)
    const uint32_t pofs = nb.piece_offset(piece);
#pragma unroll 1
    for (int u0 = 0; u0 < UNITS; u0 += W / PARTS) {   // sum j: part j % PARTS of unit u0 + j / PARTS
      v2u idx[W];
      int n[W], most = 0;
      uint32_t own[W];
#pragma unroll
      for (int j = 0; j < W; ++j) {
        const int row = first_row + (u0 + j / PARTS) * RC + (ln >> LR);
        if (PARTS == 2 && j % 2 == 1) {
          idx[j] = idx[j - 1];
          n[j] = n[j - 1];
        } else if (RC == 16) {
          idx[j] = t_idx;
          n[j] = t_n;
        } else {
          idx[j].x = (uint32_t)__shfl((int)t_idx.x, row + 16 * g, 64);
          idx[j].y = (uint32_t)__shfl((int)t_idx.y, row + 16 * g, 64);
          n[j] = RC == 1 ? __builtin_amdgcn_readlane(t_n, row) : __shfl(t_n, row, 64);
        }
        most = max(most, n[j]);
        own[j] = 0u;
        if (self)
          own[j] = __builtin_amdgcn_raw_buffer_load_b32(
              r_own, v_own, own_unit_offset((uint32_t)(first_row + (u0 + j / PARTS) * RC), hv * 256u + j % PARTS * nb.part, (uint32_t)ldx, own_size), 0);
      }
      // The first block in up to three steps, each with all of its loads in flight: wide rows are few
      // neighbours of many bytes from HBM, narrow ones more neighbours from the caches.  Few tiles of wide rows are bound by the
      // round trips instead and request at once what any row of the unit has, 4, 8 or 16 entries.  us, in steps, here, and always
      // all 16: 300 columns on 15221 rows, 14 neighbours, in front of two layers 44.5, 43.0 and 42.8; 700 on 24576 rows
      // of a power-law graph 66.4, 65.2 and 68.7, 2 neighbours 53.7, 52.6 and 56.5.  129 to 256 columns: launch_one().
      constexpr int K1 = P >= 16 ? 1 : 2;            // 4 K1 entries of every row, then up to 8, then all 16
      constexpr bool ONE = WPT == 4 && MODE != kGatherSums && (P >= 32 || (P >= 16 && WAVES == 4));
      constexpr int XK = ONE ? 4 : 2;
      v4i acc[W], x[W][XK];
      const bool five = K1 == 1 && __builtin_amdgcn_ballot_w64(most > 4) != 0ull, nine = __builtin_amdgcn_ballot_w64(most > 8) != 0ull;
      auto entries = [&](int k, int to) {
#pragma unroll
        for (int j = 0; j < W; ++j) x[j][to] = nb.load(list_entry(idx[j], k), pofs + j % PARTS * nb.part);
      };
      auto add = [&](int k) {
#pragma unroll
        for (int j = 0; j < W; ++j) acc[j] = mfma_i8(ident, x[j][k], acc[j]);
      };
#pragma unroll
      for (int k = 0; k < K1; ++k) entries(k, k);
      if (five) entries(1, 1);
      if constexpr (ONE) {
        if (nine) {
          entries(2, 2);
          entries(3, 3);
        }
      }
      all_in_flight<K1 != 1 || ONE>();
      // (the own row, and 128 for every code that is code - 128)
#pragma unroll
      for (int j = 0; j < W; ++j) {
        const int bias = p.x_offset * (n[j] + self);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[j][r] = bias + (int)(int8_t)(own[j] >> (8 * r));
      }
#pragma unroll
      for (int k = 0; k < K1; ++k) add(k);
      if (five) add(1);
      if (nine) {
        if constexpr (!ONE) {
          entries(2, 0);
          entries(3, 1);
          all_in_flight<K1 != 1>();
        }
        add(XK - 2);
        add(XK - 1);
      }
      // further blocks, a block's entries requested beside the products of the one in front
      if (__builtin_amdgcn_ballot_w64(most > kListBlock) != 0ull) {
        auto more = [&](int base) {
#pragma unroll
          for (int j = 0; j < W; ++j) {
            idx[j] = (v2u){~0u, ~0u};
            const int64_t row = row0 + first_row + (u0 + j / PARTS) * RC + (ln >> LR);
            if (n[j] > base) idx[j] = *reinterpret_cast<const v2u*>(p.rest + row * p.rest_cap + (base - kListBlock) + 4 * g);
          }
        };
        more(kListBlock);
#pragma unroll 1
        for (int base = kListBlock; __builtin_amdgcn_ballot_w64(most > base) != 0ull; base += kListBlock) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
              for (int j = 0; j < W; ++j) x[j][k] = nb.load(list_entry(idx[j], 2 * h + k), pofs + j % PARTS * nb.part);
            if (h == 1) more(base + kListBlock);
            all_in_flight<K1 != 1 || ONE>();
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
              for (int j = 0; j < W; ++j) acc[j] = mfma_i8(ident, x[j][k], acc[j]);
          }
#pragma unroll
          for (int j = 0; j < W; ++j) settle(acc[j]);
        }
      }
      if constexpr (MODE == kGatherSums) {
#pragma unroll
        for (int j = 0; j < W; ++j) {
          const int row = row0 + first_row + (u0 + j) * RC + (ln >> LR);
          if (row < p.rows && n[j] >= 0) emit_sums(p, row, 16 * piece + 4 * g, acc[j]);
        }
        continue;
      }
      const int at = parts ? piece & 15 : piece;
      uint8_t* const to = yb + (at >> 2) * 1024 + (at & 3) * 16 + 4 * g;
      if constexpr (PARTS == 2) {
#pragma unroll
        for (int j = 0; j < W; j += 2) {
          uint32_t c[4], lo, hi;
#pragma unroll
          for (int r = 0; r < 4; ++r) c[r] = (uint32_t)acc[j][r] + ((uint32_t)acc[j + 1][r] << 8);
          wide_codes(p, c, lo, hi);
          if (P <= 4 || piece < 4 * n_ks) {
            uint32_t* const word = reinterpret_cast<uint32_t*>(to + (first_row + (u0 + j / 2) * RC + (ln >> LR)) * 64);
            word[0] = kept_codes(p, lo, 16 * piece + 4 * g);
            word[n_ks * 256] = kept_codes(p, hi, 16 * piece + 4 * g);
          }
        }
      } else {
        uint32_t c[W][4], d[W];
#pragma unroll
        for (int j = 0; j < W; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) c[j][r] = (uint32_t)acc[j][r];
        pack_codes_words(c, q, d);
        if (P <= 4 || piece < 4 * n_ks) {
#pragma unroll
          for (int j = 0; j < W; ++j)
            *reinterpret_cast<uint32_t*>(to + (first_row + (u0 + j) * RC + (ln >> LR)) * 64) = kept_codes(p, d[j], 16 * piece + 4 * g);
        }
      }
    }
    if (HV > 1 && parts) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the lanes read each other's codes
      add_products<LT, MODE>(p, lds, yb, 4 * hv, min(4 * hv + 4, n_ks), 0, row_sums, z, rs, lane);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }

  // ---- 3 --------------------------------------------------------------------------------------------
  if constexpr (MODE == kGatherSums) return;
  if (HV > 1 && parts) {
    emit_tile<LT, MODE>(p, lds, row0, out_ok, 0, z, rs, rl, lane);
    return;
  }
  if (WPT != 1) __syncthreads();
  else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if constexpr (PARTS == 2) finish_wide_tile<MODE>(p, lds, yb, row0, out_ok, WPT == 1 ? 0 : wave, WPT == 1 ? 1 : 4, rl, lane);
  else finish_tile<LT, MODE>(p, lds, yb, row0, out_ok, WPT == 1 ? 0 : wave, WPT == 1 ? LT : 4, rl, lane);
}

// WAVES: per SIMD, at least, which bounds the registers of a wave.  49 to 64 columns have 97 or 98 with all of their loads in
// flight, which is four waves, and 96 with five; the others have as many waves either way, or lose with fewer registers
// (256 -> 64 -> 64 on 65536 rows 51.2 us, with 96 registers 52.9).  Five where there are more workgroups than four waves hold.
// Four and five, us, five layers of 64: 65536 rows (1024 workgroups) 55.4 and 59.7, 98304 75.6 and 75.1, 131072 88.9 and 88.1;
// of a power-law graph, 131072 rows 94.4 and 92.5, 262144 148.8 and 135, 524288 248 and 225.
// 129 to 256 columns of which four waves share a tile: the whole first block at once and four waves up to three workgroups per
// compute unit, in steps with 80 registers and six waves beyond.  200 -> 200 -> 64, 2 and 14 neighbours, us: 3584 rows (224
// workgroups) in steps 25.4 and 28.1, at once 25.5 and 27.4; 12288 (768) 28.1 and 32.4, at once 28.3 and 32.2; 16384 (1024)
// 31.5 and 36.2, at once 31.3 and 36.5; 24576 (1536) 38.1 and 45.6, at once 47.3 and 52.6.
template <int LP, int WPT, int LT, int MODE, int PARTS, int WAVES = 4>
qgtc_status launch_one(const GatherParams& p, size_t lds, hipStream_t stream) {
  if constexpr (PARTS == 1 && WAVES == 4 && (WPT == 1 ? LP == 2 : LP == 4 && MODE != kGatherSums)) {
    if (p.nblocks > (WPT == 1 ? 4u : 3u) * (unsigned)device_compute_units()) return launch_one<LP, WPT, LT, MODE, PARTS, WPT == 1 ? 5 : 6>(p, lds, stream);
  }
  static OncePerDevice once;
  if (!allow_lds(once, reinterpret_cast<const void*>(&gather_layer_kernel<LP, WPT, LT, MODE, PARTS, WAVES>), lds)) return QGTC_ERR_HIP;
  hipLaunchKernelGGL((gather_layer_kernel<LP, WPT, LT, MODE, PARTS, WAVES>), dim3((unsigned)p.n_heavy_wg + xcd_deal_grid(p.nblocks, p.run_shift)), dim3(256),
                     lds, stream, p);
  return launch_status();
}

template <int LP, int MODE, int PARTS>
qgtc_status launch_pieces(const GatherParams& p, bool share, size_t lds, hipStream_t stream) {
  if constexpr (LP >= 2) {
    if (share) return launch_one<LP, 4, 1, MODE, PARTS>(p, lds, stream);
  }
  if constexpr (MODE == kGatherSums || PARTS == 2) return launch_one<LP, 1, 1, MODE, PARTS>(p, lds, stream);
  else return p.n_nt > 1 ? launch_one<LP, 1, 4, MODE, 1>(p, lds, stream) : launch_one<LP, 1, 1, MODE, 1>(p, lds, stream);
}

}  // namespace

template <int MODE, int PARTS>
qgtc_status gather_launch(const GatherParams& p, bool share, size_t lds, hipStream_t stream) {
  const int pieces = p.ldx / (16 * PARTS);
  if (pieces <= 1) return launch_pieces<0, MODE, PARTS>(p, share, lds, stream);
  if (pieces <= 2) return launch_pieces<1, MODE, PARTS>(p, share, lds, stream);
  if (pieces <= 4) return launch_pieces<2, MODE, PARTS>(p, share, lds, stream);
  if (pieces <= 8) return launch_pieces<3, MODE, PARTS>(p, share, lds, stream);
  if (pieces <= 16) return launch_pieces<4, MODE, PARTS>(p, share, lds, stream);
  if constexpr (PARTS == 2) return launch_pieces<5, MODE, PARTS>(p, share, lds, stream);
  else return pieces <= 32 ? launch_pieces<5, MODE, PARTS>(p, share, lds, stream) : launch_pieces<6, MODE, PARTS>(p, share, lds, stream);
}

}  // namespace qgtc
