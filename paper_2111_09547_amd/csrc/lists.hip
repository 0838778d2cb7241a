// Neighbour lists of a packed adjacency: zero-tile jumping (Section 4.3 of the paper) down to the
// single entry, for graphs of a few neighbours per node.  Like the tile map, they are laid out once
// per adjacency and read by every layer; one pass over A makes both, and the degrees.
#include "lists_of.h"

namespace qgtc {
namespace {

// A wave per 16 rows reads them from A.  What bounds it is the latency of its loads and the loops over the bits; 8 MiB of A
// (65536 rows of 1024 bits, 8 bits each) are read once.
__global__ __launch_bounds__(256) void lists_kernel(const ListParams p) {
  __shared__ __attribute__((aligned(16))) uint16_t lists[4][16][kListMax];
  __shared__ uint32_t heavy[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = ((int)blockIdx.x * 4 + wave) * 16 + (lane & 15);
  const uint32_t* const row = p.A + (int64_t)(r < p.rows ? r : 0) * p.lda;
  lists_of(p, blockIdx.x, lists[wave], heavy, [&](int c) { return r < p.rows ? *reinterpret_cast<const uint4*>(row + 4 * c) : make_uint4(0u, 0u, 0u, 0u); });
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

namespace qgtc {
qgtc_status list_params(const qgtc_bits* A, const qgtc_neighbours* n, const qgtc_tile_map* map, ListParams* to) {
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
  *to = p;
  return QGTC_OK;
}
}  // namespace qgtc

extern "C" qgtc_status qgtc_build_neighbours(const qgtc_bits* A, const qgtc_neighbours* n, const qgtc_tile_map* map, void* stream) {
  ListParams p;
  const qgtc_status st = list_params(A, n, map, &p);
  if (st != QGTC_OK || A->rows == 0) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope prof(QGTC_KERNEL_TILE_MAP, s);
  hipLaunchKernelGGL(lists_kernel, dim3((unsigned)cdiv(A->rows, 64)), dim3(256), 0, s, p);
  return launch_status();
}
