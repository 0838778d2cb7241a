// What lays out neighbour lists from the words of A: lists.hip reads them from memory, pack.hip has just made them.
#pragma once
#include "lists.h"

namespace qgtc {

struct ListParams {
  const uint32_t* A;
  int64_t lda;
  int32_t rows;
  int32_t n128;              // 128-bit pieces of a row
  int32_t rest_cap;
  uint16_t* first;
  uint16_t* rest;
  uint8_t* heavy_cnt;
  uint64_t* heavy;
  int32_t* deg;
  int32_t* map_deg;          // the tile map's part (NULL: none)
  int32_t* row_cnt;
  int32_t* col_idx;
  int32_t n_tile_cols, tile_shift;   // tiles per 128-bit piece: 1 << tile_shift
};

// Checks of qgtc_build_neighbours, and its parameters.
qgtc_status list_params(const qgtc_bits* A, const qgtc_neighbours* n, const qgtc_tile_map* map, ListParams* to);

namespace {

__device__ __forceinline__ int list_at(int e) { return (e & ~15) + 4 * (e & 3) + ((e >> 2) & 3); }

// Lists, degrees and tiles of the 64 rows of workgroup `block`, a wave per 16 of them: lane <-> (row = lane % 16, one of four
// 128-bit pieces = lane / 16).  A row is read once, 16 pieces of it in flight together: piece(c) is the lane's row's piece c
// (zeros behind the last row), all read in front of the first entry that is written where there are at most 16.  Each lane
// puts the positions of its bits into the row's list in LDS (lists: the wave's), behind those of the lanes in front of it.
// heavy: four words of LDS, not those of the lists.
template <class Piece>
__device__ __forceinline__ void lists_of(const ListParams& p, unsigned block, uint16_t (*lists)[kListMax], uint32_t* heavy, Piece piece) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tr = (int)block * 4 + wave;
  const int r = tr * 16 + (lane & 15), g = lane >> 4;
  const bool r_ok = r < p.rows;
  uint16_t* const list = lists[lane & 15];
  int count = 0, tiles = 0;                          // entries of the row so far; tiles of the map
  for (int c0 = 0; c0 < p.n128; c0 += 16) {
    uint4 v[4];
    unsigned long long words = 0ull;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + 4 * u + g;
      v[u] = make_uint4(0u, 0u, 0u, 0u);
      if (c < p.n128) v[u] = piece(c);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // (the pieces may lie where the entries go)
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (c0 + 4 * u >= p.n128) continue;            // (uniform)
      const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
      const int mine = __builtin_popcount(w[0]) + __builtin_popcount(w[1]) + __builtin_popcount(w[2]) + __builtin_popcount(w[3]);
      const int s1 = __shfl_up(mine, 16, 64), s2 = __shfl_up(mine, 32, 64), s3 = __shfl_up(mine, 48, 64);
      int at = count + (g > 0 ? s1 : 0) + (g > 1 ? s2 : 0) + (g > 2 ? s3 : 0);
      count = __shfl(at + mine, 48 + (lane & 15), 64);
      const int k0 = (c0 + 4 * u + g) * 128;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint32_t m = w[i];
        while (m) {
          if (at < kListMax) list[list_at(at)] = (uint16_t)(k0 + 32 * i + __builtin_ctz(m));
          ++at;
          m &= m - 1u;
        }
      }
      if (p.row_cnt) {                               // (uniform) bit 16 u + j: word j of the four pieces holds a bit
        unsigned long long some = 0ull;              // four words of a piece at bits 16 piece ..
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          unsigned long long b = __builtin_amdgcn_ballot_w64(w[i] != 0u);
          b |= b >> 8;
          b |= b >> 4;
          b |= b >> 2;
          b |= b >> 1;
          some |= (b & 0x0001000100010001ull) << i;
        }
        words |= ((some | some >> 12 | some >> 24 | some >> 36) & 0xffffull) << (16 * u);
      }
    }
    if (p.row_cnt) {
      // the tile map's list of the 16 rows: a lane per word, the first of a tile writes it (a loop over words whose first
      // lane stores: a mini-batch of 8192 rows packed in 11.0 us, here 10.0)
      if (p.tile_shift < 2) words |= words >> 1;
      if (p.tile_shift < 1) words |= words >> 2;
      const int sub = 4 >> p.tile_shift, tile = (c0 * 4 + lane) / sub;   // words per tile
      const bool kept = (words >> lane & 1ull) != 0ull && (lane & (sub - 1)) == 0 && tile < p.n_tile_cols;
      const unsigned long long all = __builtin_amdgcn_ballot_w64(kept);
      if (kept) p.col_idx[(int64_t)tr * p.n_tile_cols + tiles + __builtin_popcountll(all & ((1ull << lane) - 1ull))] = tile;
      tiles += __builtin_popcountll(all);
    }
  }
  if (p.row_cnt && lane == 0 && tr * 16 < p.rows) p.row_cnt[tr] = tiles;
  const uint32_t many = (uint32_t)__builtin_amdgcn_ballot_w64(count > kListLight) & 0xffffu;
  if (lane == 0) heavy[wave] = many;
  const int whole = min((max(count, 1) + kListBlock - 1) / kListBlock * kListBlock, kListMax);   // whole blocks
  for (int e = count + g; e < whole; e += 4) list[list_at(e)] = kListNone;
  __syncthreads();                                   // (the lanes of a row also read each other's entries)
  if (threadIdx.x == 0) {
    const uint64_t m = (uint64_t)heavy[0] | (uint64_t)heavy[1] << 16 | (uint64_t)heavy[2] << 32 | (uint64_t)heavy[3] << 48;
    p.heavy[block] = m;
    p.heavy_cnt[block] = (uint8_t)__builtin_popcountll(m);
  }
  if (!r_ok) return;
  if (g == 0) {
    p.deg[r] = count;
    if (p.map_deg) p.map_deg[r] = count;
  }
  if (g < 2) *reinterpret_cast<uint4*>(p.first + (int64_t)r * kListBlock + 8 * g) = *reinterpret_cast<const uint4*>(list + 8 * g);
  const int kept = min(whole, kListBlock + p.rest_cap);
  for (int e = kListBlock + 8 * g; e < kept; e += 32)
    *reinterpret_cast<uint4*>(p.rest + (int64_t)r * p.rest_cap + (e - kListBlock)) = *reinterpret_cast<const uint4*>(list + e);
}

}  // namespace
}  // namespace qgtc
