// Bandwidth-optimized subgraph packing (Section 4.6 of the paper), host side: the
// adjacency and the node features of a batch are quantized and packed into bit
// planes on the CPU, side by side in ONE buffer, so that a single transfer of
// low-bit data crosses the PCIe link instead of dense fp32 matrices in several
// transfers.  Same layouts, same Eq. (2) arithmetic (fp32, separately rounded
// operations) as the device packing in pack.hip, so both give the same words.
// Plain C++; nothing here touches the GPU.
#include "qgtc_internal.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <thread>
#include <vector>

#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
#include <immintrin.h>
#endif

namespace qgtc {
namespace {

struct HostPack {
  const void* src;
  int src_dtype;
  int64_t ld_src;
  int32_t rows, cols, nbits;
  uint32_t* dst;
  int64_t ld, ps;
  float lo, inv;
  uint32_t qmax;
  float qmaxf;
};

template <int SRC>
inline uint32_t host_code(const HostPack& p, int64_t idx) {
  if constexpr (SRC == QGTC_SRC_F32) {
    const float x = reinterpret_cast<const float*>(p.src)[idx];
    const float d = x - p.lo;                       // Eq. (2), as quantize_f32 on the device
    const float t = std::floor(d * p.inv);
    if (!(t > 0.0f)) return 0u;
    if (t >= p.qmaxf) return p.qmax;
    return (uint32_t)t;
  } else if constexpr (SRC == QGTC_SRC_U8) {
    return (uint32_t)reinterpret_cast<const uint8_t*>(p.src)[idx] & p.qmax;
  } else {
    return reinterpret_cast<const uint32_t*>(p.src)[idx] & p.qmax;
  }
}

#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
// The lowest bits of 32 bytes as a word: bit 0 of every byte moves to bit 7, which is what movemask takes.
inline uint32_t low_bits_sse2(const uint8_t* b) {
  const __m128i lo = _mm_loadu_si128(reinterpret_cast<const __m128i*>(b)), hi = _mm_loadu_si128(reinterpret_cast<const __m128i*>(b + 16));
  return (uint32_t)_mm_movemask_epi8(_mm_slli_epi16(lo, 7)) | (uint32_t)_mm_movemask_epi8(_mm_slli_epi16(hi, 7)) << 16;
}
void low_bits_row(const uint8_t* row, uint32_t* out, int words) {
  for (int w = 0; w < words; ++w) out[w] = low_bits_sse2(row + 32 * w);
}
__attribute__((target("avx2"))) void low_bits_row_avx2(const uint8_t* row, uint32_t* out, int words) {
  for (int w = 0; w < words; ++w)
    out[w] = (uint32_t)_mm256_movemask_epi8(_mm256_slli_epi16(_mm256_loadu_si256(reinterpret_cast<const __m256i*>(row + 32 * w)), 7));
}
bool has_avx2() { return __builtin_cpu_supports("avx2") != 0; }
bool has_avx512() { return __builtin_cpu_supports("avx512f") != 0; }
#else
// Eight bytes at a time: the lowest bit of byte k goes to bit k of the top byte of
// (x & 0x01..01) * 0x0102040810204080.
void low_bits_row(const uint8_t* row, uint32_t* out, int words) {
  for (int w = 0; w < words; ++w) {
    uint32_t word = 0u;
    for (int k = 0; k < 4; ++k) {
      uint64_t x;
      std::memcpy(&x, row + w * 32 + k * 8, 8);
      word |= (uint32_t)(((x & 0x0101010101010101ull) * 0x0102040810204080ull) >> 56) << (8 * k);
    }
    out[w] = word;
  }
}
#endif

// The adjacency: one bit from each of 32 bytes.
void pack_left_rows_u8_1bit(const HostPack& p, int r0, int r1) {
  const uint8_t* src = reinterpret_cast<const uint8_t*>(p.src);
  auto whole = low_bits_row;
#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
  if (has_avx2()) whole = low_bits_row_avx2;
#endif
  for (int r = r0; r < r1; ++r) {
    const uint8_t* row = src + (int64_t)r * p.ld_src;
    uint32_t* out = p.dst + (int64_t)r * p.ld;
    const int full = p.cols / 32;
    whole(row, out, full);
    for (int64_t w = full; w < p.ld; ++w) {
      uint32_t word = 0u;
      for (int b = 0; b < 32 && w * 32 + b < p.cols; ++b) word |= (uint32_t)(row[w * 32 + b] & 1u) << b;
      out[w] = word;
    }
  }
}

// LEFT: rows [r0, r1); bit b of word w of a row <-> column 32 w + b; all ld words written.
template <int SRC>
void pack_left_rows(const HostPack& p, int r0, int r1) {
  if (SRC == QGTC_SRC_U8 && p.nbits == 1) {
    pack_left_rows_u8_1bit(p, r0, r1);
    return;
  }
  uint32_t codes[32];
  for (int r = r0; r < r1; ++r) {
    for (int64_t w = 0; w < p.ld; ++w) {
      const int c0 = (int)(w * 32);
      const int n = std::max(0, std::min(32, p.cols - c0));
      for (int b = 0; b < n; ++b) codes[b] = host_code<SRC>(p, (int64_t)r * p.ld_src + c0 + b);
      for (int pl = 0; pl < p.nbits; ++pl) {
        uint32_t word = 0u;
        for (int b = 0; b < n; ++b) word |= ((codes[b] >> pl) & 1u) << b;
        p.dst[(int64_t)pl * p.ps + (int64_t)r * p.ld + w] = word;
      }
    }
  }
}

// RIGHT: word rows [w0, w1); bit b of word (kw, c) <-> row 32 kw + b.  Columns [c_from, cols).
template <int SRC>
void pack_right_words_any(const HostPack& p, int w0, int w1, int c_from) {
  const int cols = p.cols - c_from;
  if (cols <= 0) return;
  std::vector<uint32_t> words((size_t)p.nbits * cols);
  std::vector<uint32_t> codes((size_t)cols);
  for (int kw = w0; kw < w1; ++kw) {
    std::fill(words.begin(), words.end(), 0u);
    const int n = std::min(32, p.rows - kw * 32);
    for (int b = 0; b < n; ++b) {                   // walk the source row by row (contiguous)
      const int64_t base = (int64_t)(kw * 32 + b) * p.ld_src + c_from;
      for (int c = 0; c < cols; ++c) codes[c] = host_code<SRC>(p, base + c);
      for (int pl = 0; pl < p.nbits; ++pl) {        // plain loops over the columns: vectorizable
        uint32_t* wp = words.data() + (size_t)pl * cols;
        for (int c = 0; c < cols; ++c) wp[c] |= ((codes[c] >> pl) & 1u) << b;
      }
    }
    for (int pl = 0; pl < p.nbits; ++pl)
      std::copy(words.begin() + (size_t)pl * cols, words.begin() + (size_t)(pl + 1) * cols,
                p.dst + (int64_t)pl * p.ps + (int64_t)kw * p.ld + c_from);
  }
}

#if !defined(__HIP_DEVICE_COMPILE__)
// fp32 to at most 8 bits, 16 columns at a time: the codes of rows r, r + 8, r + 16, r + 24 become the
// bytes of word r of their column, and three rounds of masked swaps between the eight words
// transpose its four 8 x 8 bit matrices at once into the words of the planes (as planes_word_to_codes
// does on the device; the transposition is its own inverse).  Bound by the source: 2 M values in
// 0.4 ms on one thread, where a test of the type, a floor and a walk over the planes per value took 2.6.
constexpr int kVec = 16;
typedef float VecF __attribute__((vector_size(4 * kVec), aligned(4)));
typedef int32_t VecI __attribute__((vector_size(4 * kVec)));
typedef uint32_t VecU __attribute__((vector_size(4 * kVec)));
typedef uint32_t VecUStore __attribute__((vector_size(4 * kVec), aligned(4)));

template <int SH>
inline __attribute__((always_inline)) void swap_rows(VecU& x, VecU& y, uint32_t m) {
  const VecU nx = (x & ~(m << SH)) | ((y & m) << SH);
  const VecU ny = (y & ~m) | ((x >> SH) & m);
  x = nx;
  y = ny;
}

inline __attribute__((always_inline)) void pack_right_small(const HostPack& p, int w0, int w1) {
  const VecF lo = VecF{} + p.lo, inv = VecF{} + p.inv, most = VecF{} + p.qmaxf, zero = VecF{};
  const int whole = p.cols / kVec * kVec;
  for (int kw = w0; kw < w1; ++kw) {
    const int n = std::min(32, p.rows - kw * 32);
    for (int c = 0; c < whole; c += kVec) {
      const float* src = reinterpret_cast<const float*>(p.src) + (int64_t)kw * 32 * p.ld_src + c;
      VecU a[8];
      for (int r = 0; r < 8; ++r) {
        a[r] = VecU{};
        for (int b = 0; b < 4; ++b) {
          if (8 * b + r >= n) continue;
          VecF t = (*reinterpret_cast<const VecF*>(src + (int64_t)(8 * b + r) * p.ld_src) - lo) * inv;
          t = t > zero ? t : zero;                   // (a NaN: code 0)
          t = t < most ? t : most;
          a[r] |= (VecU)__builtin_convertvector(t, VecI) << (8 * b);   // truncation is the floor here
        }
      }
      for (int r = 0; r < 4; ++r) swap_rows<4>(a[r], a[r + 4], 0x0f0f0f0fu);
      for (int r = 0; r < 8; r += 4) {
        swap_rows<2>(a[r], a[r + 2], 0x33333333u);
        swap_rows<2>(a[r + 1], a[r + 3], 0x33333333u);
      }
      for (int r = 0; r < 8; r += 2) swap_rows<1>(a[r], a[r + 1], 0x55555555u);
      uint32_t* dst = p.dst + (int64_t)kw * p.ld + c;
      for (int pl = 0; pl < p.nbits; ++pl) *reinterpret_cast<VecUStore*>(dst + (int64_t)pl * p.ps) = a[pl];
    }
  }
}
void pack_right_small_any(const HostPack& p, int w0, int w1) { pack_right_small(p, w0, w1); }
#if defined(__x86_64__)
__attribute__((target("avx2"))) void pack_right_small_avx2(const HostPack& p, int w0, int w1) { pack_right_small(p, w0, w1); }
__attribute__((target("avx512f"))) void pack_right_small_avx512(const HostPack& p, int w0, int w1) { pack_right_small(p, w0, w1); }
#endif
#endif

template <int SRC>
void pack_right_words(const HostPack& p, int w0, int w1) {
  int done = 0;
#if !defined(__HIP_DEVICE_COMPILE__)
  if (SRC == QGTC_SRC_F32 && p.nbits <= 8) {
    auto small = pack_right_small_any;
#if defined(__x86_64__)
    if (has_avx2()) small = pack_right_small_avx2;
    if (has_avx512()) small = pack_right_small_avx512;
#endif
    small(p, w0, w1);
    done = p.cols / kVec * kVec;
  }
#endif
  pack_right_words_any<SRC>(p, w0, w1, done);
}

// Rows (LEFT) or word rows (RIGHT) [a, b) of an operand.
void pack_range(const HostPack& p, bool left, int a, int b) {
  switch (p.src_dtype) {
    case QGTC_SRC_F32: return left ? pack_left_rows<QGTC_SRC_F32>(p, a, b) : pack_right_words<QGTC_SRC_F32>(p, a, b);
    case QGTC_SRC_U8: return left ? pack_left_rows<QGTC_SRC_U8>(p, a, b) : pack_right_words<QGTC_SRC_U8>(p, a, b);
    default: return left ? pack_left_rows<QGTC_SRC_I32>(p, a, b) : pack_right_words<QGTC_SRC_I32>(p, a, b);
  }
}

// One or two operands, in pieces of some 128 KiB of source that the threads take one after the
// other, so that a thread that starts late takes fewer.
struct HostJob {
  HostPack p[2];
  bool left[2];
  int n = 0;                                         // operands
  int items[2], step[2], pieces[2];                  // rows or word rows, of a piece, pieces
  int64_t worth = 0;                                 // threads that pay, in 1/16
  std::atomic<int> next{0};

  void add(const HostPack& pack, bool is_left) {
    p[n] = pack;
    left[n] = is_left;
    items[n] = is_left ? pack.rows : cdiv(pack.rows, 32);
    const int64_t row = (int64_t)pack.cols * (pack.src_dtype == QGTC_SRC_U8 ? 1 : 4) * (is_left ? 1 : 32);
    step[n] = (int)std::max<int64_t>(1, (128 << 10) / row);
    pieces[n] = cdiv(items[n], step[n]);
    // A thread takes as long to start as 4 MiB of a vectorized loop (16 MiB of adjacency and 8 MiB of features: one
    // thread 510 us, two 328, four 176, eight 189, sixteen 347), or 512 KiB of another.
    const bool fast = pack.nbits <= 8 && (is_left ? pack.src_dtype == QGTC_SRC_U8 && pack.nbits == 1 : pack.src_dtype == QGTC_SRC_F32);
    worth += 16 * row * items[n] / (fast ? 4 << 20 : 512 << 10);
    ++n;
  }
  int all() const { return pieces[0] + (n > 1 ? pieces[1] : 0); }
  void work() {
    for (int k; (k = next.fetch_add(1, std::memory_order_relaxed)) < all();) {
      const int o = k < pieces[0] ? 0 : 1, at = (o == 0 ? k : k - pieces[0]) * step[o];
      pack_range(p[o], left[o], at, at + std::min(step[o], items[o] - at));
    }
  }
  // Threads [a, b): the first is this one, which starts the others with half of what is left each (a thread
  // takes some 15 us to start, one after the other 16 of them more than the work).
  void run(int a, int b) {
    std::vector<std::thread> started;
    while (b - a > 1) {
      const int mid = a + (b - a) / 2;
      try {
        started.emplace_back([this, mid, b] { run(mid, b); });
      } catch (...) {                                // no more threads to be had: the others do it
        break;
      }
      b = mid;
    }
    work();
    for (auto& t : started) t.join();
  }
  void start(int threads) { run(0, (int)std::max<int64_t>(1, std::min<int64_t>(threads, std::min<int64_t>(all(), 1 + worth / 16)))); }
};

qgtc_status host_operand(const void* src, int32_t src_dtype, int32_t rows, int32_t cols, int64_t ld_src, const qgtc_quant* q,
                         const qgtc_bits* dst, HostPack* out) {
  if (!src || !dst) return QGTC_ERR_NULL;
  if (dst->layout != QGTC_LEFT && dst->layout != QGTC_RIGHT) return QGTC_ERR_UNSUPPORTED;
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
  HostPack& p = *out;
  p = HostPack{};
  p.src = src;
  p.src_dtype = src_dtype;
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
  return QGTC_OK;
}

int host_threads(int threads) { return threads == 0 ? (int)std::max(1u, std::thread::hardware_concurrency()) : threads; }

}  // namespace
}  // namespace qgtc

using namespace qgtc;

extern "C" qgtc_status qgtc_pack_bits_host(const void* src, int32_t src_dtype, int32_t rows, int32_t cols,
                                           int64_t ld_src, const qgtc_quant* q, const qgtc_bits* dst,
                                           int32_t threads) {
  HostPack p;
  const qgtc_status st = host_operand(src, src_dtype, rows, cols, ld_src, q, dst, &p);
  if (st != QGTC_OK) return st;
  if (threads < 0) return QGTC_ERR_SHAPE;
  if (rows == 0 || cols == 0) return QGTC_OK;
  HostJob job;
  job.add(p, dst->layout == QGTC_LEFT);
  job.start(host_threads(threads));
  return QGTC_OK;
}

extern "C" qgtc_status qgtc_pack_batch_host(const qgtc_host_operand* ops, int32_t n, int32_t threads) {
  if (!ops) return QGTC_ERR_NULL;
  if (n < 1 || n > 2 || threads < 0) return QGTC_ERR_SHAPE;
  HostPack p[2];
  for (int i = 0; i < n; ++i) {
    const qgtc_status st = host_operand(ops[i].src, ops[i].src_dtype, ops[i].rows, ops[i].cols, ops[i].ld_src, ops[i].q, ops[i].dst, &p[i]);
    if (st != QGTC_OK) return st;
  }
  HostJob job;
  for (int i = 0; i < n; ++i)
    if (p[i].rows > 0 && p[i].cols > 0) job.add(p[i], ops[i].dst->layout == QGTC_LEFT);
  if (job.n > 0) job.start(host_threads(threads));
  return QGTC_OK;
}

extern "C" size_t qgtc_compound_layout(const size_t* bytes, int32_t n, size_t* offsets) {
  if (n < 0 || (n > 0 && (!bytes || !offsets))) return 0;
  size_t total = 0;
  for (int i = 0; i < n; ++i) {
    offsets[i] = total;
    total += (bytes[i] + 255) / 256 * 256;
  }
  return total;
}
