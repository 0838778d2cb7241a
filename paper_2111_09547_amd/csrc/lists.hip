// Neighbour lists of a packed adjacency: zero-tile jumping (Section 4.3 of the paper) down to the
// single entry, for graphs of a few neighbours per node.  Like the tile map, they are laid out once
// per adjacency and read by every layer; one pass over A makes both, and the degrees.
#include "lists.h"

namespace qgtc {
namespace {

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

__device__ __forceinline__ int list_at(int e) { return (e & ~15) + 4 * (e & 3) + ((e >> 2) & 3); }

// A wave per 16 rows, lane <-> (row = lane % 16, one of four 128-bit pieces = lane / 16).  A row is read
// once, 16 pieces of it in flight together; each lane puts the positions of its bits into the row's
// list in LDS, behind those of the lanes in front of it.  What bounds it is the latency of its
// loads and the loops over the bits; 8 MiB of A (65536 rows of 1024 bits, 8 bits each) are read once.
__global__ __launch_bounds__(256) void lists_kernel(const ListParams p) {
  __shared__ __attribute__((aligned(16))) uint16_t lists[4][16][kListMax];
  __shared__ uint32_t heavy[4];                      // the waves' heavy rows
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int tr = blockIdx.x * 4 + wave;
  const int r = tr * 16 + (lane & 15), g = lane >> 4;
  const bool r_ok = r < p.rows;
  const uint32_t* row = p.A + (int64_t)(r_ok ? r : 0) * p.lda;
  uint16_t* const list = lists[wave][lane & 15];
  int count = 0, tiles = 0;                          // entries of the row so far; tiles of the map
  for (int c0 = 0; c0 < p.n128; c0 += 16) {
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + 4 * u + g;
      v[u] = make_uint4(0u, 0u, 0u, 0u);
      if (r_ok && c < p.n128) v[u] = *reinterpret_cast<const uint4*>(row + 4 * c);
    }
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
      if (p.row_cnt) {                               // (uniform) the tile map's list of the 16 rows
        unsigned long long b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) b[i] = __builtin_amdgcn_ballot_w64(w[i] != 0u);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          uint32_t bits = 0u;                        // words of the piece that hold a bit
#pragma unroll
          for (int i = 0; i < 4; ++i) bits |= ((b[i] >> (16 * k)) & 0xffffull) != 0ull ? 1u << i : 0u;
          const int sub = 4 >> p.tile_shift;         // words per tile
          for (int c = 0; c < 1 << p.tile_shift; ++c) {
            const int tile = ((c0 + 4 * u + k) << p.tile_shift) + c;
            if (((bits >> (c * sub)) & ((1u << sub) - 1u)) != 0u && tile < p.n_tile_cols) {
              if (lane == 0) p.col_idx[(int64_t)tr * p.n_tile_cols + tiles] = tile;
              ++tiles;
            }
          }
        }
      }
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
    p.heavy[blockIdx.x] = m;
    p.heavy_cnt[blockIdx.x] = (uint8_t)__builtin_popcountll(m);
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

int rest_cap_of(int cols) {
  const int more = cdiv(cols, kListBlock) * kListBlock - kListBlock;
  return more < kListMax - kListBlock ? more : kListMax - kListBlock;
}
bool lists_cover(const qgtc_bits* A) {
  return A->cols >= 1 && A->cols < kListNone && (A->block_rows > 0 || A->cols == A->rows);
}
size_t align16(size_t v) { return (v + 15) & ~(size_t)15; }

}  // namespace

qgtc_status check_neighbours(const qgtc_neighbours* n, const qgtc_bits* A) {
  if (!n->deg || !n->heavy || !n->heavy_cnt || !n->first || (n->rest_cap > 0 && !n->rest)) return QGTC_ERR_NULL;
  if (!lists_cover(A)) return QGTC_ERR_UNSUPPORTED;
  if (n->rows != A->rows || n->cols != A->cols || n->block_rows != A->block_rows || n->rest_cap != rest_cap_of(A->cols))
    return QGTC_ERR_SHAPE;
  // as wide as the kernels read them
  if ((((uintptr_t)n->first | (uintptr_t)n->rest | (uintptr_t)n->heavy_cnt) & 15u) != 0) return QGTC_ERR_ALIGN;
  if (((uintptr_t)n->heavy & 7u) != 0 || ((uintptr_t)n->deg & 3u) != 0) return QGTC_ERR_ALIGN;
  return QGTC_OK;
}

}  // namespace qgtc

using namespace qgtc;

// deg, masks, counts (whole 16-byte pieces), first blocks, the others
extern "C" size_t qgtc_neighbours_bytes(const qgtc_bits* A) {
  if (!A || check_adjacency(A) != QGTC_OK || A->rows < 1 || !lists_cover(A)) return 0;
  const size_t rows = (size_t)A->rows, groups = (size_t)cdiv(A->rows, kListGroup);
  return align16(rows * 4) + align16(groups * 8) + align16(groups) + rows * (size_t)(kListBlock + rest_cap_of(A->cols)) * 2;
}

extern "C" qgtc_status qgtc_neighbours_carve(qgtc_neighbours* n, void* buffer, const qgtc_bits* A) {
  if (!n || !buffer || !A) return QGTC_ERR_NULL;
  qgtc_status st = check_adjacency(A);
  if (st != QGTC_OK) return st;
  if (A->rows < 1 || !lists_cover(A)) return QGTC_ERR_UNSUPPORTED;
  if (((uintptr_t)buffer & 15u) != 0) return QGTC_ERR_ALIGN;
  n->rows = A->rows;
  n->cols = A->cols;
  n->block_rows = A->block_rows;
  n->rest_cap = rest_cap_of(A->cols);
  const size_t rows = (size_t)A->rows, groups = (size_t)cdiv(A->rows, kListGroup);
  char* b = reinterpret_cast<char*>(buffer);
  n->deg = reinterpret_cast<int32_t*>(b);
  b += align16(rows * 4);
  n->heavy = reinterpret_cast<uint64_t*>(b);
  b += align16(groups * 8);
  n->heavy_cnt = reinterpret_cast<uint8_t*>(b);
  b += align16(groups);
  n->first = reinterpret_cast<uint16_t*>(b);
  b += rows * kListBlock * 2;
  n->rest = reinterpret_cast<uint16_t*>(b);
  return QGTC_OK;
}

extern "C" qgtc_status qgtc_build_neighbours(const qgtc_bits* A, const qgtc_neighbours* n, const qgtc_tile_map* map, void* stream) {
  if (!A || !n) return QGTC_ERR_NULL;
  qgtc_status st = check_adjacency(A);
  if (st != QGTC_OK) return st;
  st = check_neighbours(n, A);
  if (st != QGTC_OK) return st;
  ListParams p{};
  if (map) {
    if (!map->row_cnt || !map->col_idx || !map->deg) return QGTC_ERR_NULL;
    if (map->tile_rows != 16 || (map->tile_kbits != 32 && map->tile_kbits != 64 && map->tile_kbits != 128)) return QGTC_ERR_UNSUPPORTED;
    if (map->n_tile_rows != cdiv(A->rows, 16) || map->n_tile_cols != cdiv(A->cols, map->tile_kbits)) return QGTC_ERR_SHAPE;
    p.map_deg = map->deg;
    p.row_cnt = map->row_cnt;
    p.col_idx = map->col_idx;
    p.n_tile_cols = map->n_tile_cols;
    p.tile_shift = map->tile_kbits == 128 ? 0 : (map->tile_kbits == 64 ? 1 : 2);
  }
  if (A->rows == 0) return QGTC_OK;
  p.A = A->data;
  p.lda = A->ld_words;
  p.rows = A->rows;
  p.n128 = cdiv(A->cols, 128);
  p.rest_cap = n->rest_cap;
  p.first = n->first;
  p.rest = n->rest;
  p.heavy = n->heavy;
  p.heavy_cnt = n->heavy_cnt;
  p.deg = n->deg;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope prof(QGTC_KERNEL_TILE_MAP, s);
  hipLaunchKernelGGL(lists_kernel, dim3((unsigned)cdiv(A->rows, 64)), dim3(256), 0, s, p);
  return launch_status();
}
