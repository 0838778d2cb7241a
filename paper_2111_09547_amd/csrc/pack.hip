// Quantize + bit-decompose + pack ("Tensor.to_bit"), decode ("Tensor.to_val")
// and the value sums of packed operands.  Eq. (2) and the 3D-stacked bit
// compression of Section 4.2 of the paper, for gfx950.  All of these are
// streaming kernels bound by HBM bandwidth.
#include "gather.h"
#include "lists_of.h"

namespace qgtc {
namespace {

struct PackParams {
  const void* src;
  int64_t ld_src;
  int32_t rows, cols;
  int32_t nbits;
  uint32_t* dst;
  int64_t ld, ps;       // words
  float lo, inv;        // Eq. (2), fp32 sources only
  uint32_t qmax;
  float qmaxf;
  uint32_t flip;        // QGTC_LEFT_BYTES: on every word (0x80808080: codes - 128)
  int32_t shift;        // RIGHT_BYTES of wider codes: their bits from here on
};

template <int SRC> struct src_type { using type = uint32_t; };
template <> struct src_type<QGTC_SRC_F32> { using type = float; };
template <> struct src_type<QGTC_SRC_U8> { using type = uint8_t; };

// Raw element (the load) and its code (Eq. (2) or masking) are kept apart so
// that many loads can be in flight before the first conversion.
template <int SRC>
__device__ __forceinline__ typename src_type<SRC>::type fetch_raw(const PackParams& p, int64_t idx) {
  return reinterpret_cast<const typename src_type<SRC>::type*>(p.src)[idx];
}

template <int SRC>
__device__ __forceinline__ uint32_t to_code(const PackParams& p, typename src_type<SRC>::type v) {
  if constexpr (SRC == QGTC_SRC_F32) {
    return quantize_f32(v, p.lo, p.inv, p.qmax, p.qmaxf);
  } else {
    return (uint32_t)v & p.qmax;
  }
}

template <int SRC>
__device__ __forceinline__ uint32_t fetch(const PackParams& p, int64_t idx) {
  return to_code<SRC>(p, fetch_raw<SRC>(p, idx));
}

// RIGHT layout: 32 consecutive ROWS of one column share a word.
// thread <-> (column c, word row w); the 32 loads of a thread are each
// coalesced across the threads of the wave (consecutive columns).
template <int SRC>
__global__ __launch_bounds__(256) void pack_right_kernel(const PackParams p) {
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int w_row = blockIdx.y * 4 + (threadIdx.x >> 6);
  const int n_wr = (p.rows + 31) >> 5;
  if (c >= p.cols || w_row >= n_wr) return;
  // all 32 loads of the word are issued before the first one is used
  typename src_type<SRC>::type raw[32];
#pragma unroll
  for (int b = 0; b < 32; ++b) {
    const int r = min(w_row * 32 + b, p.rows - 1);      // clamped: no branch around the load
    raw[b] = fetch_raw<SRC>(p, (int64_t)r * p.ld_src + c);
  }
  uint32_t q[32];
#pragma unroll
  for (int b = 0; b < 32; ++b) q[b] = (w_row * 32 + b < p.rows) ? to_code<SRC>(p, raw[b]) : 0u;
  // 8 planes at a time: the codes of 8 rows are an 8 x 8 bit matrix (a byte per row)
  // whose transpose has a byte per plane; four of them make the 32 rows of a word
  for (int p0 = 0; p0 < p.nbits; p0 += 8) {
    uint32_t L[4], H[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      uint32_t lo = 0u, hi = 0u;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        lo |= ((q[8 * g + k] >> p0) & 0xffu) << (8 * k);
        hi |= ((q[8 * g + 4 + k] >> p0) & 0xffu) << (8 * k);
      }
      transpose_bits_8x8(lo, hi);
      L[g] = lo;
      H[g] = hi;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int sh = 8 * (i & 3);
      uint32_t w = 0u;
#pragma unroll
      for (int g = 0; g < 4; ++g) w |= (((i < 4 ? L[g] : H[g]) >> sh) & 0xffu) << (8 * g);
      if (p0 + i < p.nbits) p.dst[(int64_t)(p0 + i) * p.ps + (int64_t)w_row * p.ld + c] = w;
    }
  }
}

// LEFT layout: 32 consecutive COLUMNS of one row share a word.
// One wave per row; lane <-> column inside a 64-column chunk, so the loads are
// coalesced and a ballot over the lanes yields two finished words.  The words
// of 32 chunks are gathered lane by lane and stored 256 bytes at a time.
// Every word up to ld (the zero padding included) is written.
template <int SRC>
__global__ __launch_bounds__(256) void pack_left_kernel(const PackParams p) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= p.rows) return;                       // whole wave
  const int n_words = (int)p.ld;
  for (int pl = 0; pl < p.nbits; ++pl) {
    uint32_t* drow = p.dst + (int64_t)pl * p.ps + (int64_t)r * p.ld;
    for (int w0 = 0; w0 < n_words; w0 += 64) {   // 64 words = 2048 columns per pass
      uint32_t mine = 0u;
      const int n_chunks = min(32, (n_words - w0 + 1) >> 1);
      for (int ch = 0; ch < n_chunks; ++ch) {
        const int c = (w0 + 2 * ch) * 32 + lane;
        uint32_t bit = 0u;
        if (c < p.cols) bit = (fetch<SRC>(p, (int64_t)r * p.ld_src + c) >> pl) & 1u;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(bit != 0u);
        if (lane == 2 * ch) mine = (uint32_t)m;
        if (lane == 2 * ch + 1) mine = (uint32_t)(m >> 32);
      }
      if (w0 + lane < n_words) drow[w0 + lane] = mine;
    }
  }
}

// Fast path for a 0/1 byte matrix into one plane (the adjacency): every lane
// loads 16 consecutive bytes, squeezes them into 16 bits, neighbouring lanes
// merge their halves with a DPP shift, and the even lanes store finished words.
// Needs cols and ld_src multiples of 16 and a 16-byte aligned source.
__device__ __forceinline__ uint32_t squeeze4(uint32_t d) {
  uint32_t t = d & 0x01010101u;     // bit 0 of each byte
  t |= t >> 7;                      // bytes 0,1 -> bits 0,1 ; bytes 2,3 -> bits 16,17
  t |= t >> 14;                     // -> bits 0..3
  return t & 0xfu;
}

// A unit is 1024 columns of one row (64 lanes x 16 bytes); a wave takes UNITS units, all
// of their loads in flight together.  Measured on 64 MiB to 1 GiB of input with 1, 2, 4
// and 8 units per wave and grids capped at 2048 to 8192 workgroups or not at all: two units
// and one wave per pair of units is the fastest or level everywhere (5.0 - 5.7 TB/s of
// read + written bytes from 128 MiB on).
constexpr int kU8Units = 2;

template <int UNITS>
__global__ __launch_bounds__(256) void pack_left_u8_kernel(const PackParams p) {
  const int lane = threadIdx.x & 63;
  const int n_words = (int)p.ld;
  const int n_pass = (n_words + 31) >> 5;          // units per row
  const int64_t n_units = (int64_t)p.rows * n_pass;
  const int64_t wave_id = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
  const int64_t step = (int64_t)gridDim.x * 4 * UNITS;
  // (row, unit within the row) of the wave's first unit and of the stride: one division
  // each per wave, then additions only
  int64_t r0 = wave_id * UNITS / n_pass;
  int q0 = (int)(wave_id * UNITS % n_pass);
  const int64_t step_r = step / n_pass;
  const int step_q = (int)(step % n_pass);
  const uint8_t* src = reinterpret_cast<const uint8_t*>(p.src);
  for (int64_t u0 = wave_id * UNITS; u0 < n_units; u0 += step) {
    uint4 v[UNITS];
    int64_t r = r0;
    int q = q0;
#pragma unroll
    for (int k = 0; k < UNITS; ++k) {
      const int c = q * 1024 + lane * 16;
      v[k] = make_uint4(0u, 0u, 0u, 0u);
      if (r < p.rows && c < p.cols) v[k] = *reinterpret_cast<const uint4*>(src + r * p.ld_src + c);
      if (++q == n_pass) { q = 0; ++r; }
    }
    r = r0;
    q = q0;
#pragma unroll
    for (int k = 0; k < UNITS; ++k) {
      const int w = q * 32 + (lane >> 1);
      const uint32_t h = squeeze4(v[k].x) | (squeeze4(v[k].y) << 4) | (squeeze4(v[k].z) << 8) |
                         (squeeze4(v[k].w) << 12);
      // odd lane's half moves down to the even lane (wave shift left by one lane)
      const uint32_t up = (uint32_t)__shfl_down((int)h, 1, 64);
      if ((lane & 1) == 0 && r < p.rows && w < n_words) p.dst[r * p.ld + w] = h | (up << 16);
      if (++q == n_pass) { q = 0; ++r; }
    }
    r0 += step_r;
    q0 += step_q;
    if (q0 >= n_pass) { q0 -= n_pass; ++r0; }
  }
}

// RIGHT_BYTES: thread (tile nt, step ks, lane l) writes the 16 codes of column
// 16 nt + l % 16, rows 64 ks + 16 (l / 16) .. + 15, as bytes (see qgtc.h).
template <int SRC>
__device__ __forceinline__ void pack_bytes_of(const PackParams& p, int n_nt, int n_ks, int idx) {
  const int lane = idx & 63;
  const int ks = (idx >> 6) % n_ks;
  const int nt = (idx >> 6) / n_ks;
  if (nt >= n_nt) return;
  const int col = nt * 16 + (lane & 15);
  const int k0 = ks * 64 + (lane >> 4) * 16;
  typename src_type<SRC>::type raw[16];
#pragma unroll
  for (int b = 0; b < 16; ++b) {
    const bool ok = col < p.cols && k0 + b < p.rows;
    raw[b] = fetch_raw<SRC>(p, ok ? (int64_t)(k0 + b) * p.ld_src + col : 0);
  }
  uint32_t d[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int b = 0; b < 16; ++b) {
    const bool ok = col < p.cols && k0 + b < p.rows;
    const uint32_t code = ok ? (to_code<SRC>(p, raw[b]) >> p.shift) & 0xffu : 0u;
    d[b >> 2] |= code << (8 * (b & 3));
  }
  uint4* dst = reinterpret_cast<uint4*>(reinterpret_cast<uint8_t*>(p.dst) + (int64_t)idx * 16);
  if (p.nbits == 8) {
    dst[p.ps / 4] = make_uint4((d[0] >> 7) & 0x01010101u, (d[1] >> 7) & 0x01010101u,
                               (d[2] >> 7) & 0x01010101u, (d[3] >> 7) & 0x01010101u);
    dst[0] = make_uint4(d[0] & 0x7f7f7f7fu, d[1] & 0x7f7f7f7fu, d[2] & 0x7f7f7f7fu, d[3] & 0x7f7f7f7fu);
  } else {
    dst[0] = make_uint4(d[0], d[1], d[2], d[3]);
  }
}

template <int SRC>
__global__ __launch_bounds__(256) void pack_bytes_kernel(const PackParams p, int n_nt, int n_ks) {
  pack_bytes_of<SRC>(p, n_nt, n_ks, blockIdx.x * 256 + threadIdx.x);
}

// The weights of several layers at once (RIGHT_BYTES from fp32), and the column sums of the codes of one of
// them.  Each is a few KiB: what a launch of its own took was the launch.
constexpr int kWeightJobs = 16;
struct WeightsParams {
  PackParams w[kWeightJobs];
  int32_t n_nt[kWeightJobs], n_ks[kWeightJobs];
  int32_t end[kWeightJobs];  // first workgroup behind the job's
  int32_t n;
  int32_t sums_of;           // job whose column sums are wanted, by the workgroups behind the last job (-1: none)
  int32_t* sums;
};
__device__ __forceinline__ void pack_weights_of(const WeightsParams& jobs, int block) {
  int j = 0;
  while (j < jobs.n && block >= jobs.end[j]) ++j;
  const int lane = threadIdx.x & 63;
  if (j == jobs.n) {                                 // a wave has 16 columns, a quarter of the rows per lane
    const PackParams& p = jobs.w[jobs.sums_of];
    const int c0 = ((block - jobs.end[jobs.n - 1]) * 4 + (int)(threadIdx.x >> 6)) * 16, col = c0 + (lane & 15);
    if (c0 >= p.cols) return;
    uint32_t sum = 0u;
#pragma unroll 8
    for (int r = lane >> 4; r < p.rows; r += 4) sum += fetch<QGTC_SRC_F32>(p, (int64_t)r * p.ld_src + min(col, p.cols - 1));
    sum += (uint32_t)__shfl_xor((int)sum, 16, 64);
    sum += (uint32_t)__shfl_xor((int)sum, 32, 64);
    if (lane < 16 && col < p.cols) jobs.sums[col] = (int32_t)sum;
    return;
  }
  pack_bytes_of<QGTC_SRC_F32>(jobs.w[j], jobs.n_nt[j], jobs.n_ks[j], (block - (j > 0 ? jobs.end[j - 1] : 0)) * 256 + (int)threadIdx.x);
}
__global__ __launch_bounds__(256) void pack_weights_kernel(const WeightsParams jobs) { pack_weights_of(jobs, (int)blockIdx.x); }

// LEFT_BYTES: one code per byte, row-major; a thread writes 4 consecutive bytes.  Bound by its 4-byte loads: features of
// a width that is no multiple of four run at 4 to 5 TB/s.  The quantizer to the order of whole tiles, which those took
// before they were rows, and this one, us: 65536 x 101 10.6 and 8.9, 262144 x 101 33 and 27, x 301 101 and 82,
// x 513 171 and 141.
template <int SRC>
__global__ __launch_bounds__(256) void pack_left_bytes_kernel(const PackParams p) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;   // dword index
  const int64_t r = idx / p.ld;
  const int w = (int)(idx % p.ld);
  if (r >= p.rows) return;
  typename src_type<SRC>::type raw[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int c = w * 4 + b;
    raw[b] = fetch_raw<SRC>(p, c < p.cols ? r * p.ld_src + c : 0);
  }
  uint32_t v = 0u;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int c = w * 4 + b;
    v |= (c < p.cols ? to_code<SRC>(p, raw[b]) : 0u) << (8 * b);
  }
  p.dst[idx] = v ^ p.flip;
}

// The same where four columns are one 16-byte load (32-bit sources; cols and ld_src multiples
// of 4, aligned): bound by HBM.  A thread takes kByteWords words that lie 256 apart, so that
// every load of a wave is 1 KiB in one piece and all of them are in flight together; the
// (row, word) pairs follow from one 32-bit division and additions (rows x ld below 2^31).
// Four columns make a whole word, or padding, which is not read.  The source is not kept in the
// caches, so that the codes still are when the product reads them.  262144 x 512 fp32 (671 MB in
// and out): 119 us = 5.7 TB/s; with 4-byte loads and a 64-bit division per word, as above, the
// pass around it (two layers, update first) took 240 instead of 222 us.
constexpr int kByteWords = 4;

template <int SRC>
__device__ __forceinline__ void pack_left_bytes_wide_of(const PackParams& p, int step_r, int step_w, unsigned block) {
  const int ld = (int)p.ld;
  const unsigned idx = block * (256u * kByteWords) + threadIdx.x;
  const int r0 = (int)(idx / (unsigned)ld), w0 = (int)(idx % (unsigned)ld);
  using T = typename src_type<SRC>::type;
  typedef T Quad __attribute__((ext_vector_type(4)));
  Quad raw[kByteWords];
  int r = r0, w = w0;
#pragma unroll
  for (int k = 0; k < kByteWords; ++k) {
    // clamped to a quad that exists: no branch around the load
    const int64_t at = (int64_t)min(r, p.rows - 1) * p.ld_src + min(4 * w, p.cols - 4);
    raw[k] = __builtin_nontemporal_load(reinterpret_cast<const Quad*>(reinterpret_cast<const T*>(p.src) + at));
    r += step_r;
    w += step_w;
    if (w >= ld) { w -= ld; ++r; }
  }
  r = r0;
  w = w0;
#pragma unroll
  for (int k = 0; k < kByteWords; ++k) {
    uint32_t v = 0u;
#pragma unroll
    for (int b = 0; b < 4; ++b) v |= to_code<SRC>(p, raw[k][b]) << (8 * b);
    if (r < p.rows) p.dst[(int64_t)r * ld + w] = (4 * w < p.cols ? v : 0u) ^ p.flip;
    r += step_r;
    w += step_w;
    if (w >= ld) { w -= ld; ++r; }
  }
}

template <int SRC>
__global__ __launch_bounds__(256) void pack_left_bytes_wide_kernel(const PackParams p, int step_r, int step_w) {
  pack_left_bytes_wide_of<SRC>(p, step_r, step_w, blockIdx.x);
}

// Features and, by the first `groups` workgroups, the weights of a stack, which nothing of the features waits for:
// by itself their launch stands 7 us in front of a pass, bound by the chain of arguments, weights, codes.  The
// recorded step on 65536 nodes (five layers) 97.7 -> 92.8 us, launched one by one on 8192 nodes 58 -> 53.
__global__ __launch_bounds__(256) void pack_codes_and_weights_kernel(const WeightsParams jobs, unsigned groups, const PackParams p, int step_r,
                                                                     int step_w) {
  if (blockIdx.x < groups) pack_weights_of(jobs, (int)blockIdx.x);
  else pack_left_bytes_wide_of<QGTC_SRC_F32>(p, step_r, step_w, blockIdx.x - groups);
}

// Four columns of LEFT_BYTES are one load.
bool left_bytes_wide(const PackParams& p) {
  return (p.cols & 3) == 0 && (p.ld_src & 3) == 0 && ((uintptr_t)p.src & 15u) == 0 && (int64_t)p.rows * p.ld < (int64_t)1 << 31;
}
unsigned left_bytes_wide_groups(const PackParams& p) { return (unsigned)cdiv((int64_t)p.rows * p.ld, 256 * kByteWords); }

// A mini-batch in one launch: the adjacency from bytes with its neighbour lists and map, the weights, and the features as
// row-major codes.  Bound by HBM: 65536 rows of 1024 bytes and of 128 features, 115 MB in and out, 25.6 us = 4.5 TB/s, of
// which the lists take 4.5 beside the loads; three launches, of which the second reads back what the first wrote, 10, 13 and 8
// and their gaps (the whole step 90.4 and 83.7 us, eager batches of 8192 rows, whose launches the host bounds, 53.8 and 42.3).
// Workgroups of the lists in front: they are the longer ones (behind the features 86.3 us, among them 89.9).
struct BatchParams {
  PackParams a;              // bytes of the adjacency; a.dst: its words
  int32_t pieces;            // 16-byte pieces of a row, padding to 128 columns included
  uint32_t pieces_magic;
  ListParams lists;
  unsigned list_groups, weight_groups;
  PackParams x;
  int32_t x_step_r, x_step_w;
  WeightsParams jobs;
};

// A wave has 16 rows, whose bytes become words in LDS, kBatchLoads loads of 1 KiB in flight (4 or 16: level); the words go to memory and, from
// where they are, into the lists.
constexpr int kBatchPieces = 128;                    // of a row: 2048 columns
constexpr int kBatchLoads = 8;
__device__ __forceinline__ void pack_lists_of(const BatchParams& p, unsigned block, uint16_t (*lists)[16][kListMax], uint32_t* heavy) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row0 = ((int)block * 4 + wave) * 16;
  const int n_rows = min(p.a.rows - row0, 16);       // (none for a wave behind the last row)
  // a row's words, and 16 bytes that spread the rows over the banks
  const int stride = 2 * p.pieces + 16;
  static_assert(16 * (2 * kBatchPieces + 16) <= 16 * kListMax * 2, "the words lie where the lists will");
  uint8_t* const words = reinterpret_cast<uint8_t*>(lists[wave]);
  const uint8_t* const src = reinterpret_cast<const uint8_t*>(p.a.src) + (int64_t)row0 * p.a.ld_src;
  const int n = n_rows * p.pieces;
#pragma unroll 1
  for (int i0 = lane; i0 < n; i0 += 64 * kBatchLoads) {
    uint4 v[kBatchLoads];
    int at[kBatchLoads];
#pragma unroll
    for (int k = 0; k < kBatchLoads; ++k) {
      const unsigned i = (unsigned)min(i0 + 64 * k, n - 1);
      const int r = (int)div_by(i, (unsigned)p.pieces, p.pieces_magic), c = (int)i - r * p.pieces;
      at[k] = r * stride + 2 * c;
      v[k] = make_uint4(0u, 0u, 0u, 0u);
      if (16 * c < p.a.cols) v[k] = *reinterpret_cast<const uint4*>(src + (int64_t)r * p.a.ld_src + 16 * c);
    }
#pragma unroll
    for (int k = 0; k < kBatchLoads; ++k) {
      const uint32_t h = squeeze4(v[k].x) | (squeeze4(v[k].y) << 4) | (squeeze4(v[k].z) << 8) | (squeeze4(v[k].w) << 12);
      *reinterpret_cast<uint16_t*>(words + at[k]) = (uint16_t)h;   // (the last piece maybe several times)
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the lanes read each other's halves
  const int ld4 = (int)p.a.ld >> 2, n128 = p.lists.n128;
  for (int i = lane; i < n_rows * ld4; i += 64) {
    const int r = i / ld4, c = i - r * ld4;
    const uint4 v = c < n128 ? *reinterpret_cast<const uint4*>(words + r * stride + 16 * c) : make_uint4(0u, 0u, 0u, 0u);
    *reinterpret_cast<uint4*>(p.a.dst + (int64_t)(row0 + r) * p.a.ld + 4 * c) = v;
  }
  const int mine = lane & 15;
  lists_of(p.lists, block, lists[wave], heavy,
           [&](int c) { return mine < n_rows ? *reinterpret_cast<const uint4*>(words + mine * stride + 16 * c) : make_uint4(0u, 0u, 0u, 0u); });
}

__global__ __launch_bounds__(256) void pack_batch_kernel(const BatchParams p) {
  __shared__ __attribute__((aligned(16))) uint16_t lists[4][16][kListMax];
  __shared__ uint32_t heavy[4];
  if (blockIdx.x < p.list_groups) pack_lists_of(p, blockIdx.x, lists, heavy);
  else if (blockIdx.x < p.list_groups + p.weight_groups) pack_weights_of(p.jobs, (int)(blockIdx.x - p.list_groups));
  else pack_left_bytes_wide_of<QGTC_SRC_F32>(p.x, p.x_step_r, p.x_step_w, blockIdx.x - p.list_groups - p.weight_groups);
}

struct UnpackParams {
  const uint32_t* src;
  int64_t ld, ps;
  int32_t rows, cols, nbits, layout;
  uint32_t* dst;
  int64_t ld_dst;
};

// Planes packed along the columns, four columns of a row per item: one 16-byte store, and eight neighbouring threads read the
// same words.  A thread has ITEMS items a grid apart, whose words are in flight together.  Bound by its launch and what it
// writes; with an element and a 4-byte store per thread (unpack_kernel), and here, us: 16384 x 256 of 4 bits (18 MB,
// 3.7 at the rate of a copy) 12.8 and 7.6, of 8 bits 22.5 and 9.0, 12000 x 256 of 2 bits 8.7 and 5.8.
template <int PLANES, int ITEMS>   // PLANES: at most
__global__ __launch_bounds__(256) void unpack_left_kernel(const UnpackParams p, unsigned quads, uint32_t quad_magic, unsigned n) {
  const unsigned step = gridDim.x * 256u, i0 = blockIdx.x * 256u + threadIdx.x;
  uint32_t w[ITEMS][PLANES];
  unsigned row[ITEMS], quad[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const unsigned i = min(i0 + k * step, n - 1u);
    row[k] = div_by(i, quads, quad_magic);
    quad[k] = i - row[k] * quads;
    const uint32_t* const from = p.src + (int64_t)row[k] * p.ld + (quad[k] >> 3);
#pragma unroll
    for (int pl = 0; pl < PLANES; ++pl) {
      w[k][pl] = 0u;
      if (pl < p.nbits) w[k][pl] = from[(int64_t)pl * p.ps];
    }
  }
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (i0 + k * step >= n) return;
    const int sh = 4 * (quad[k] & 7);
    uint32_t v[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int pl = 0; pl < PLANES; ++pl)
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] |= ((w[k][pl] >> (sh + c)) & 1u) << pl;
    uint32_t* const to = p.dst + (int64_t)row[k] * p.ld_dst + 4 * quad[k];
    if (4 * (int)quad[k] + 4 <= p.cols) {
      *reinterpret_cast<uint4*>(to) = make_uint4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (4 * (int)quad[k] + c < p.cols) to[c] = v[c];
    }
  }
}

__global__ __launch_bounds__(256) void unpack_kernel(const UnpackParams p) {
  const int c = blockIdx.x * 64 + (threadIdx.x & 63);
  const int r = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (c >= p.cols || r >= p.rows) return;
  uint32_t v = 0u;
  if (p.layout == QGTC_LEFT_BYTES) {
    p.dst[(int64_t)r * p.ld_dst + c] = reinterpret_cast<const uint8_t*>(p.src)[(int64_t)r * p.ld * 4 + c];
    return;
  }
  if (p.layout == QGTC_RIGHT_BYTES) {
    const uint8_t* bytes = reinterpret_cast<const uint8_t*>(p.src);
    const int64_t off = (int64_t)(c >> 4) * p.ld * 4 + (int64_t)(r >> 6) * 1024 +
                        ((c & 15) + 16 * ((r & 63) >> 4)) * 16 + (r & 15);
    v = bytes[off];
    if (p.nbits == 8) v |= (uint32_t)bytes[p.ps * 4 + off] << 7;
    p.dst[(int64_t)r * p.ld_dst + c] = v;
    return;
  }
  for (int i = 0; i < p.nbits; ++i) {
    uint32_t word, bit;
    if (p.layout == QGTC_LEFT) {
      word = p.src[(int64_t)i * p.ps + (int64_t)r * p.ld + (c >> 5)];
      bit = c & 31;
    } else {
      word = p.src[(int64_t)i * p.ps + (int64_t)(r >> 5) * p.ld + c];
      bit = r & 31;
    }
    v |= ((word >> bit) & 1u) << i;
  }
  p.dst[(int64_t)r * p.ld_dst + c] = v;
}

// sum_p 2^p popcount(row r of plane p): one wave per row, lanes stride over words.
__global__ __launch_bounds__(256) void row_sums_kernel(const UnpackParams p, int32_t* out) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= p.rows) return;
  const int n_words = (p.cols + 31) >> 5;
  uint32_t acc = 0u;
  for (int i = 0; i < p.nbits; ++i) {
    const uint32_t* row = p.src + (int64_t)i * p.ps + (int64_t)r * p.ld;
    uint32_t cnt = 0u;
    for (int w = lane; w < n_words; w += 64) cnt += __builtin_popcount(row[w]);
    acc += cnt << i;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0) out[r] = (int32_t)acc;
}

// Same for short rows (a few words): one thread per row.
__global__ __launch_bounds__(256) void row_sums_short_kernel(const UnpackParams p, int32_t* out) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= p.rows) return;
  const int n_words = (p.cols + 31) >> 5;
  uint32_t acc = 0u;
  for (int i = 0; i < p.nbits; ++i) {
    const uint32_t* row = p.src + (int64_t)i * p.ps + (int64_t)r * p.ld;
    uint32_t cnt = 0u;
    for (int w = 0; w < n_words; ++w) cnt += __builtin_popcount(row[w]);
    acc += cnt << i;
  }
  out[r] = (int32_t)acc;
}

// sum_p 2^p popcount(column c of plane p): thread per column.
__global__ __launch_bounds__(256) void col_sums_kernel(const UnpackParams p, int32_t* out) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= p.cols) return;
  if (p.layout == QGTC_RIGHT_BYTES) {
    // bytes of column c: 16 at a time (one 16-byte load), both parts; rows past the
    // last one are stored as zeros
    const uint8_t* bytes = reinterpret_cast<const uint8_t*>(p.src);
    uint32_t sum = 0u, top = 0u;
#pragma unroll 4
    for (int r0 = 0; r0 < p.rows; r0 += 16) {
      const int64_t off = (int64_t)(c >> 4) * p.ld * 4 + (int64_t)(r0 >> 6) * 1024 +
                          ((c & 15) + 16 * ((r0 & 63) >> 4)) * 16;
      const uint4 v = *reinterpret_cast<const uint4*>(bytes + off);
      sum = __builtin_amdgcn_sad_u8(v.x, 0u, sum);
      sum = __builtin_amdgcn_sad_u8(v.y, 0u, sum);
      sum = __builtin_amdgcn_sad_u8(v.z, 0u, sum);
      sum = __builtin_amdgcn_sad_u8(v.w, 0u, sum);
      if (p.nbits == 8) {
        const uint4 h = *reinterpret_cast<const uint4*>(bytes + p.ps * 4 + off);
        top = __builtin_amdgcn_sad_u8(h.x, 0u, top);
        top = __builtin_amdgcn_sad_u8(h.y, 0u, top);
        top = __builtin_amdgcn_sad_u8(h.z, 0u, top);
        top = __builtin_amdgcn_sad_u8(h.w, 0u, top);
      }
    }
    sum += top << 7;
    out[c] = (int32_t)sum;
    return;
  }
  const int n_wr = (p.rows + 31) >> 5;
  uint32_t acc = 0u;
  for (int i = 0; i < p.nbits; ++i) {
    uint32_t cnt = 0u;
    for (int w = 0; w < n_wr; ++w) cnt += __builtin_popcount(p.src[(int64_t)i * p.ps + (int64_t)w * p.ld + c]);
    acc += cnt << i;
  }
  out[c] = (int32_t)acc;
}

template <int SRC>
qgtc_status launch_pack(const PackParams& p, int layout, hipStream_t s) {
  if (layout == QGTC_LEFT_BYTES) {
    const int64_t most = ((1ll << 31) - 1) / p.ld;   // rows of a launch, which has a thread per word and fewer than 2^32
    for (int64_t r0 = 0; r0 < p.rows; r0 += most) {
      PackParams part = p;
      part.rows = (int32_t)(p.rows - r0 < most ? p.rows - r0 : most);
      part.src = reinterpret_cast<const typename src_type<SRC>::type*>(p.src) + r0 * p.ld_src;
      part.dst = p.dst + r0 * p.ld;
      bool wide = false;
      if constexpr (SRC != QGTC_SRC_U8) {
        wide = left_bytes_wide(part);
        if (wide)
          hipLaunchKernelGGL((pack_left_bytes_wide_kernel<SRC>), dim3(left_bytes_wide_groups(part)), dim3(256), 0, s, part,
                             (int)(256 / p.ld), (int)(256 % p.ld));
      }
      if (!wide)
        hipLaunchKernelGGL((pack_left_bytes_kernel<SRC>), dim3((unsigned)cdiv((int64_t)part.rows * p.ld, 256)), dim3(256), 0, s, part);
      const qgtc_status st = launch_status();
      if (st != QGTC_OK) return st;
    }
    return QGTC_OK;
  } else if (layout == QGTC_RIGHT_BYTES) {
    const int n_nt = cdiv(p.cols, 16), n_ks = cdiv(p.rows, 64);
    hipLaunchKernelGGL((pack_bytes_kernel<SRC>), dim3((unsigned)cdiv((int64_t)n_nt * n_ks * 64, 256)), dim3(256),
                       0, s, p, n_nt, n_ks);
  } else if (layout == QGTC_RIGHT) {
    dim3 grid((unsigned)cdiv(p.cols, 64), (unsigned)cdiv(cdiv(p.rows, 32), 4));
    hipLaunchKernelGGL((pack_right_kernel<SRC>), grid, dim3(256), 0, s, p);
  } else if (SRC == QGTC_SRC_U8 && p.nbits == 1 && (p.cols & 15) == 0 && (p.ld_src & 15) == 0 &&
             ((uintptr_t)p.src & 15u) == 0) {
    const int64_t units = (int64_t)p.rows * cdiv(p.ld, 32);
    const int64_t blocks = cdiv(units, 4 * kU8Units);        // beyond 2^24 workgroups the waves loop
    hipLaunchKernelGGL(pack_left_u8_kernel<kU8Units>, dim3((unsigned)(blocks < (1 << 24) ? blocks : (1 << 24))),
                       dim3(256), 0, s, p);
  } else {
    hipLaunchKernelGGL((pack_left_kernel<SRC>), dim3((unsigned)cdiv(p.rows, 4)), dim3(256), 0, s, p);
  }
  return launch_status();
}

UnpackParams unpack_params(const qgtc_bits* m) {
  UnpackParams p{};
  p.src = m->data;
  p.ld = m->ld_words;
  p.ps = m->plane_stride_words;
  p.rows = m->rows;
  p.cols = m->cols;
  p.nbits = m->nbits;
  p.layout = m->layout;
  return p;
}

// Codes of 9 to 16 bits as rows of low bytes and behind them of high bytes, all minus 128: a thread has
// four columns.  Bound by HBM and its 4-byte loads; planes of 16 bits (pack_right_kernel) and this one, us: 65536 x 64 8.2 and
// 8.0, 262144 x 64 18.9 and 19.2, x 101 40 and 28, x 300 125 and 88, x 512 164 and 144 (805 MB in and out: 5.6 TB/s).
__global__ __launch_bounds__(256) void pack_wide_rows_kernel(const PackParams p, int quads) {
  const unsigned idx = blockIdx.x * 256u + threadIdx.x;
  const int r = (int)(idx / (unsigned)quads), c0 = 4 * (int)(idx % (unsigned)quads);
  if (r >= p.rows) return;
  float v[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = fetch_raw<QGTC_SRC_F32>(p, (int64_t)r * p.ld_src + min(c0 + k, p.cols - 1));
  uint32_t lo = 0u, hi = 0u;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t c = to_code<QGTC_SRC_F32>(p, v[k]);
    lo |= (c & 0xffu) << (8 * k);
    hi |= (c >> 8) << (8 * k);
  }
  uint32_t* const dst = p.dst + (int64_t)r * p.ld + (c0 >> 2);
  dst[0] = lo ^ 0x80808080u;
  dst[p.ld >> 1] = hi ^ 0x80808080u;
}

PackParams row_codes_params(const float* src, int64_t ld_src, int rows, int cols, const qgtc_quant* q, uint8_t* dst) {
  PackParams p{};
  p.src = src;
  p.ld_src = ld_src;
  p.rows = rows;
  p.cols = cols;
  p.nbits = q->nbits;
  p.dst = reinterpret_cast<uint32_t*>(dst);
  p.ld = row_codes_ld(cols) / 4;
  p.qmax = (1u << q->nbits) - 1u;
  p.qmaxf = (float)p.qmax;
  p.lo = (float)q->lo;
  p.inv = qgtc_quant_inv_scale(q->lo, q->hi, q->nbits);
  p.flip = row_codes_flip(q->nbits);
  return p;
}

qgtc_status check_weights(const qgtc_weight_source* ws, int n, int sums_of, const int32_t* col_sums) {
  if (!ws) return QGTC_ERR_NULL;
  if (n < 1 || sums_of >= n) return QGTC_ERR_SHAPE;
  if (sums_of >= 0 && !col_sums) return QGTC_ERR_NULL;
  for (int i = 0; i < n; ++i) {
    if (!ws[i].src || !ws[i].dst) return QGTC_ERR_NULL;
    const qgtc_status st = check_bits(ws[i].dst, QGTC_RIGHT_BYTES);
    if (st != QGTC_OK) return st;
    if (ws[i].ld_src < ws[i].dst->cols || !(ws[i].q.hi > ws[i].q.lo)) return QGTC_ERR_SHAPE;
    // (bytes 0 and 1 of codes of up to 16 bits)
    const int shift = ws[i].shift, left = ws[i].q.nbits - shift;
    if ((shift != 0 && shift != 8) || ws[i].q.nbits > 16 || ws[i].dst->nbits != (left < 8 ? left : 8)) return QGTC_ERR_BITWIDTH;
  }
  return QGTC_OK;
}

// The jobs of the weights from i0 on; their workgroups.
int weight_jobs(const qgtc_weight_source* ws, int n, int i0, int sums_of, int32_t* col_sums, WeightsParams* jobs) {
  jobs->n = n - i0 < kWeightJobs ? n - i0 : kWeightJobs;
  int groups = 0;
  for (int i = 0; i < jobs->n; ++i) {
    const qgtc_weight_source& w = ws[i0 + i];
    const qgtc_bits* dst = w.dst;
    PackParams& p = jobs->w[i];
    p.src = w.src;
    p.ld_src = w.ld_src;
    p.rows = dst->rows;
    p.cols = dst->cols;
    p.nbits = dst->nbits;
    p.dst = dst->data;
    p.ld = dst->ld_words;
    p.ps = dst->plane_stride_words;
    p.shift = w.shift;
    p.qmax = (1u << w.q.nbits) - 1u;
    p.qmaxf = (float)p.qmax;
    p.lo = (float)w.q.lo;
    p.inv = qgtc_quant_inv_scale(w.q.lo, w.q.hi, w.q.nbits);
    jobs->n_nt[i] = cdiv(p.cols, 16);
    jobs->n_ks[i] = cdiv(p.rows, 64);
    groups += cdiv((int64_t)jobs->n_nt[i] * jobs->n_ks[i] * 64, 256);
    jobs->end[i] = groups;
  }
  jobs->sums_of = sums_of >= i0 && sums_of < i0 + jobs->n ? sums_of - i0 : -1;
  jobs->sums = col_sums;
  return jobs->sums_of >= 0 ? groups + cdiv(ws[sums_of].dst->cols, 64) : groups;
}

}  // namespace

qgtc_status pack_row_codes(const float* src, int64_t ld_src, int rows, int cols, const qgtc_quant* q, uint8_t* dst,
                           hipStream_t stream) {
  const PackParams p = row_codes_params(src, ld_src, rows, cols, q, dst);
  ProfScope prof(QGTC_KERNEL_PACK, stream);
  return launch_pack<QGTC_SRC_F32>(p, QGTC_LEFT_BYTES, stream);
}

qgtc_status pack_row_codes_and_weights(const qgtc_weight_source* ws, int n, int sums_of, int32_t* col_sums, const float* src, int64_t ld_src,
                                       int rows, int cols, const qgtc_quant* q, uint8_t* dst, hipStream_t stream) {
  const qgtc_status st = check_weights(ws, n, sums_of, col_sums);
  if (st != QGTC_OK) return st;
  const PackParams p = row_codes_params(src, ld_src, rows, cols, q, dst);
  if (n > kWeightJobs || rows == 0 || cols == 0 || !left_bytes_wide(p)) {
    const qgtc_status w = qgtc_pack_weights(ws, n, sums_of, col_sums, stream);
    return w != QGTC_OK || rows == 0 || cols == 0 ? w : pack_row_codes(src, ld_src, rows, cols, q, dst, stream);
  }
  WeightsParams jobs{};
  const unsigned groups = (unsigned)weight_jobs(ws, n, 0, sums_of, col_sums, &jobs);
  ProfScope prof(QGTC_KERNEL_PACK, stream);
  hipLaunchKernelGGL(pack_codes_and_weights_kernel, dim3(groups + left_bytes_wide_groups(p)), dim3(256), 0, stream, jobs, groups, p,
                     (int)(256 / p.ld), (int)(256 % p.ld));
  return launch_status();
}

qgtc_status pack_wide_rows(const float* src, int64_t ld_src, int rows, int cols, const qgtc_quant* q, uint8_t* dst, hipStream_t stream) {
  PackParams p = row_codes_params(src, ld_src, rows, cols, q, dst);
  p.ld *= 2;                                         // words of both bytes
  const int quads = (int)(p.ld / 2);
  ProfScope prof(QGTC_KERNEL_PACK, stream);
  hipLaunchKernelGGL(pack_wide_rows_kernel, dim3((unsigned)cdiv((int64_t)rows * quads, 256)), dim3(256), 0, stream, p, quads);
  return launch_status();
}

}  // namespace qgtc

using namespace qgtc;

extern "C" qgtc_status qgtc_pack_bits(const void* src, int32_t src_dtype, int32_t rows, int32_t cols,
                                      int64_t ld_src, const qgtc_quant* q, const qgtc_bits* dst,
                                      void* stream) {
  if (!src || !dst) return QGTC_ERR_NULL;
  qgtc_status st = check_bits(dst, dst->layout);
  if (st != QGTC_OK) return st;
  if (rows != dst->rows || cols != dst->cols || ld_src < cols) return QGTC_ERR_SHAPE;
  if (src_dtype != QGTC_SRC_F32 && src_dtype != QGTC_SRC_U8 && src_dtype != QGTC_SRC_I32)
    return QGTC_ERR_UNSUPPORTED;
  if (src_dtype == QGTC_SRC_F32) {
    if (!q) return QGTC_ERR_NULL;
    if (q->nbits != dst->nbits) return QGTC_ERR_BITWIDTH;
    if (!(q->hi > q->lo)) return QGTC_ERR_SHAPE;
  }
  if (dst->layout == QGTC_RIGHT && dst->ld_words < cols) return QGTC_ERR_SHAPE;
  if (rows == 0 || cols == 0) return QGTC_OK;

  PackParams p{};
  p.src = src;
  p.ld_src = ld_src;
  p.rows = rows;
  p.cols = cols;
  p.nbits = dst->nbits;
  p.dst = dst->data;
  p.ld = dst->ld_words;
  p.ps = dst->plane_stride_words;
  p.qmax = dst->nbits >= 32 ? 0xffffffffu : ((1u << dst->nbits) - 1u);
  p.qmaxf = (float)p.qmax;
  if (src_dtype == QGTC_SRC_F32) {
    p.lo = (float)q->lo;
    p.inv = (float)((double)(1ull << q->nbits) / (q->hi - q->lo));
  }
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope prof(QGTC_KERNEL_PACK, s);
  switch (src_dtype) {
    case QGTC_SRC_F32: return launch_pack<QGTC_SRC_F32>(p, dst->layout, s);
    case QGTC_SRC_U8: return launch_pack<QGTC_SRC_U8>(p, dst->layout, s);
    default: return launch_pack<QGTC_SRC_I32>(p, dst->layout, s);
  }
}

extern "C" qgtc_status qgtc_pack_weights(const qgtc_weight_source* ws, int32_t n, int32_t sums_of, int32_t* col_sums, void* stream) {
  const qgtc_status st = check_weights(ws, n, sums_of, col_sums);
  if (st != QGTC_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  for (int i0 = 0; i0 < n; i0 += kWeightJobs) {
    WeightsParams jobs{};
    const int groups = weight_jobs(ws, n, i0, sums_of, col_sums, &jobs);
    if (groups == 0) continue;
    ProfScope prof(QGTC_KERNEL_PACK, s);
    hipLaunchKernelGGL(pack_weights_kernel, dim3((unsigned)groups), dim3(256), 0, s, jobs);
    if (launch_status() != QGTC_OK) return QGTC_ERR_HIP;
  }
  return QGTC_OK;
}

extern "C" qgtc_status qgtc_pack_batch(const uint8_t* a_src, int64_t ld_a, const qgtc_bits* A, const qgtc_neighbours* lists,
                                       const qgtc_tile_map* map, const qgtc_weight_source* ws, int32_t n, int32_t sums_of,
                                       int32_t* col_sums, const float* x, int32_t x_cols, int64_t ld_x, const qgtc_quant* q, void* buffer,
                                       size_t buffer_bytes, void* stream) {
  if (!a_src || !A) return QGTC_ERR_NULL;
  BatchParams b{};
  qgtc_status st = list_params(A, lists, map, &b.lists);
  if (st != QGTC_OK) return st;
  if (ld_a < A->cols) return QGTC_ERR_SHAPE;
  st = check_weights(ws, n, sums_of, col_sums);
  if (st != QGTC_OK) return st;
  if (x) {
    st = check_row_codes(x, A->rows, x_cols, ld_x, q, buffer, buffer_bytes);
    if (st != QGTC_OK) return st;
  }
  const int rows = A->rows;
  if (x) b.x = row_codes_params(x, ld_x, rows, x_cols, q, reinterpret_cast<uint8_t*>(buffer));
  // One launch where the bytes are read 16 at a time, a row's words fit its list, and the features are read 16 bytes at a time;
  // else one each.
  bool one = rows > 0 && (A->cols & 15) == 0 && A->cols <= 16 * kBatchPieces && (ld_a & 15) == 0 && ((uintptr_t)a_src & 15u) == 0 &&
                   n <= kWeightJobs && (!x || (x_cols > 0 && left_bytes_wide(b.x)));
  // Recorded, where a launch costs the host nothing, few long rows are split over more workgroups by launches of their own: the
  // 64 rows of a workgroup are 96 KiB and more here, which one compute unit reads, and others idle.  New inputs at every
  // replay, 20 columns of features, us of a step in one launch and in three: 8192 rows of 2048 36.7 and 31.0, 7680 of
  // 1536 32.3 and 28.5, 16384 of 2048 38.5 and 35.0, 32768 43.9 and 43.9; 8192 of 1024 25.9 and 26.1.  With 128 columns, whose
  // codes are beside the rows, 8192 of 2048 37.8 and 38.8; not recorded 31.7 and 36.6.
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  if (one && A->cols > 1024 && cdiv(rows, 64) <= device_compute_units() && (!x || 16 * (int64_t)x_cols < A->cols)) {
    hipStreamCaptureStatus recorded = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &recorded) != hipSuccess) (void)hipGetLastError();
    one = recorded == hipStreamCaptureStatusNone;
  }
  if (!one) {
    if (x) st = qgtc_stack_input_and_weights(x, rows, x_cols, ld_x, q, buffer, buffer_bytes, ws, n, sums_of, col_sums, stream);
    else st = qgtc_pack_weights(ws, n, sums_of, col_sums, stream);
    if (st == QGTC_OK) st = qgtc_pack_bits(a_src, QGTC_SRC_U8, rows, A->cols, ld_a, nullptr, A, stream);
    return st == QGTC_OK ? qgtc_build_neighbours(A, lists, map, stream) : st;
  }
  b.a.src = a_src;
  b.a.ld_src = ld_a;
  b.a.rows = rows;
  b.a.cols = A->cols;
  b.a.dst = A->data;
  b.a.ld = A->ld_words;
  b.pieces = 8 * b.lists.n128;
  b.pieces_magic = div_magic(b.pieces);
  b.list_groups = (unsigned)cdiv(rows, 64);
  b.weight_groups = (unsigned)weight_jobs(ws, n, 0, sums_of, col_sums, &b.jobs);
  unsigned groups = b.list_groups + b.weight_groups;
  if (x) {
    b.x_step_r = (int32_t)(256 / b.x.ld);
    b.x_step_w = (int32_t)(256 % b.x.ld);
    groups += left_bytes_wide_groups(b.x);
  }
  ProfScope prof(QGTC_KERNEL_PACK, s);
  hipLaunchKernelGGL(pack_batch_kernel, dim3(groups), dim3(256), 0, s, b);
  return launch_status();
}

extern "C" qgtc_status qgtc_unpack_bits(const qgtc_bits* src, uint32_t* dst, int64_t ld_dst, void* stream) {
  if (!src || !dst) return QGTC_ERR_NULL;
  qgtc_status st = check_bits(src, src->layout);
  if (st != QGTC_OK) return st;
  if (ld_dst < src->cols) return QGTC_ERR_SHAPE;
  if (src->rows == 0 || src->cols == 0) return QGTC_OK;
  UnpackParams p = unpack_params(src);
  p.dst = dst;
  p.ld_dst = ld_dst;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope prof(QGTC_KERNEL_PACK, s);
  const int64_t quads = cdiv(p.cols, 4), items = quads * p.rows;
  if (p.layout == QGTC_LEFT && p.nbits <= 8 && (ld_dst & 3) == 0 && ((uintptr_t)dst & 15u) == 0 && items < (int64_t)1 << 30) {
    const uint32_t magic = div_magic((int)quads);
    // (four items where every compute unit still has four workgroups)
    const bool four = items >= (int64_t)4 * 4 * 256 * device_compute_units();
    const dim3 grid((unsigned)cdiv(items, four ? 1024 : 256));
    auto kernel = four ? (p.nbits <= 4 ? unpack_left_kernel<4, 4> : unpack_left_kernel<8, 4>)
                       : (p.nbits <= 4 ? unpack_left_kernel<4, 1> : unpack_left_kernel<8, 1>);
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, p, (unsigned)quads, magic, (unsigned)items);
    return launch_status();
  }
  dim3 grid((unsigned)cdiv(p.cols, 64), (unsigned)cdiv(p.rows, 4));
  hipLaunchKernelGGL(unpack_kernel, grid, dim3(256), 0, s, p);
  return launch_status();
}

extern "C" qgtc_status qgtc_row_sums(const qgtc_bits* m, int32_t* out, void* stream) {
  if (!m || !out) return QGTC_ERR_NULL;
  qgtc_status st = check_bits(m, QGTC_LEFT);
  if (st != QGTC_OK) return st;
  if (m->rows == 0) return QGTC_OK;
  UnpackParams p = unpack_params(m);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope prof(QGTC_KERNEL_SUMS, s);
  if (p.cols <= 256)
    hipLaunchKernelGGL(row_sums_short_kernel, dim3((unsigned)cdiv(p.rows, 256)), dim3(256), 0, s, p, out);
  else
    hipLaunchKernelGGL(row_sums_kernel, dim3((unsigned)cdiv(p.rows, 4)), dim3(256), 0, s, p, out);
  return launch_status();
}

extern "C" qgtc_status qgtc_col_sums(const qgtc_bits* m, int32_t* out, void* stream) {
  if (!m || !out) return QGTC_ERR_NULL;
  qgtc_status st = check_bits(m, m->layout == QGTC_RIGHT_BYTES ? QGTC_RIGHT_BYTES : QGTC_RIGHT);
  if (st != QGTC_OK) return st;
  if (m->cols == 0) return QGTC_OK;
  UnpackParams p = unpack_params(m);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  ProfScope prof(QGTC_KERNEL_SUMS, s);
  hipLaunchKernelGGL(col_sums_kernel, dim3((unsigned)cdiv(p.cols, 256)), dim3(256), 0, s, p, out);
  return launch_status();
}
