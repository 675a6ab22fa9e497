// Host-side quantizer and packer of libvbq (layout version 1, include/vbq.h).
//
// vbq_pack quantizes each 64-weight group as in paper section 3.1 (Eq. (1) for
// b in {2,4,8}, sign times absmean for b = 1) and writes the packed blob;
// vbq_pack_codes packs levels that were quantized elsewhere.  Both run in two
// passes over row tiles on host threads: count the groups of each width per
// unit, then write every section at its final offset.
//
// What bounds it: a group's arithmetic (the 1-bit mean's chain of 64 dependent
// additions, 64 double divisions at b >= 2) and, for small matrices, starting
// threads.  So the divisions, the rounding and the sign masks are AVX2 where the
// processor has it (the same operations in double, the same results), codes are
// packed by shifts on 64-bit words, and a thread is started per
// 4096 groups.  2048 x 8192, mixed widths, 16 processors: 3.57 -> 1.07 ms (one
// thread of a 2.7 GHz Xeon: 66 -> 21 ms; 501 x 448: 1.2 -> 0.3 ms).

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <thread>
#include <vector>

// (VBQ_PACK_PORTABLE: without the AVX2 code, for tests)
#if defined(__x86_64__) && !defined(VBQ_PACK_PORTABLE)
#define VBQ_PACK_AVX2
#include <immintrin.h>
#endif

#include "vbq_layout.hpp"

using namespace vbq;

namespace {

struct Counts {
  std::vector<uint32_t> per_unit;  // [units][4]
};

// Run fn(t) for every tile t on up to n_threads host threads (0: as many as the
// processor has, one per `grain` of the `work` groups at most; starting one
// costs about as much as a thousand groups).  The calling thread is one of them.
template <class F>
void parallel_tiles(int64_t T, uint32_t n_threads, int64_t work, int64_t grain, F&& fn) {
  int64_t nt = n_threads;
  if (nt == 0) {
    const unsigned hw = std::thread::hardware_concurrency();
    nt = std::min<int64_t>(hw ? hw : 1, work / grain + 1);
  }
  nt = std::min<int64_t>(std::min<int64_t>(nt, 64), T);
  if (nt <= 1) {
    for (int64_t t = 0; t < T; ++t) fn(t);
    return;
  }
  std::atomic<int64_t> next{0};
  auto loop = [&] {
    for (int64_t t; (t = next.fetch_add(1)) < T;) fn(t);
  };
  std::vector<std::thread> pool;
  pool.reserve((size_t)nt);
  for (int64_t i = 1; i < nt; ++i) {
    try {
      pool.emplace_back(loop);
    } catch (...) {
      break;  // no further thread to be had: the ones there are do the rest
    }
  }
  loop();
  for (auto& th : pool) th.join();
}

constexpr int64_t kCountGrain = 1 << 20;  // groups per thread: counting (0.5 ns a group)
constexpr int64_t kPackGrain = 1 << 12;   // quantizing and packing (20-60 ns a group)

void record_error(std::atomic<int>& err, vbq_status s) {
  int expected = VBQ_OK;
  err.compare_exchange_strong(expected, (int)s);
}

// One group of a width as a count of its class in a 16-bit field (a unit has at
// most 8192 groups); widths outside {1, 2, 4, 8} count in none.
struct ClassCounts {
  uint64_t one[256] = {};
  ClassCounts() {
    for (int c = 0; c < 4; ++c) one[1 << c] = 1ull << (16 * c);
  }
};

// Count the groups of each class per unit and validate the bit map.
vbq_status count_units(const Geometry& g, const uint8_t* bits, uint32_t n_threads, Counts* out) {
  static const ClassCounts kCounts;
  out->per_unit.resize((size_t)g.units * 4);
  std::atomic<int> err{VBQ_OK};
  parallel_tiles(g.T, n_threads, g.N * g.G, kCountGrain, [&](int64_t t) {
    if (err.load(std::memory_order_relaxed) != VBQ_OK) return;
    int64_t rows = g.tile_rows(t);
    for (int64_t k = 0; k < g.U; ++k) {
      uint32_t* cnt = &out->per_unit[(size_t)(t * g.U + k) * 4];
      int64_t j0 = k * g.C, cols = g.chunk_cols(k);
      uint64_t sum = 0;
      for (int64_t rl = 0; rl < rows; ++rl) {
        const uint8_t* brow = bits + (t * g.R + rl) * g.G + j0;
        for (int64_t jl = 0; jl < cols; ++jl) sum += kCounts.one[brow[jl]];
      }
      int64_t valid = 0;
      for (int c = 0; c < 4; ++c) valid += cnt[c] = (uint32_t)((sum >> (16 * c)) & 0xFFFFu);
      if (valid != rows * cols) {
        record_error(err, VBQ_ERR_BITS);
        return;
      }
    }
  });
  return (vbq_status)err.load();
}

// Prefix sums of the counts into per-unit starting entries, and the totals.
vbq_status unit_starts(const Geometry& g, const Counts& cnt, std::vector<uint32_t>* starts,
                       int64_t n_entries[4]) {
  starts->assign((size_t)(g.units + 1) * 4, 0);
  uint64_t run[4] = {0, 0, 0, 0};
  for (int64_t u = 0; u <= g.units; ++u) {
    for (int c = 0; c < 4; ++c) {
      if (run[c] > 0xFFFFFFFFull) return VBQ_ERR_UNSUPPORTED;
      (*starts)[(size_t)u * 4 + c] = (uint32_t)run[c];
      if (u < g.units) run[c] += cnt.per_unit[(size_t)u * 4 + c];
    }
  }
  for (int c = 0; c < 4; ++c) n_entries[c] = (int64_t)run[c];
  if ((uint64_t)g.wmap_words > 0xFFFFFFFFull) return VBQ_ERR_UNSUPPORTED;
  return VBQ_OK;
}

// Word offset of unit (t, k) in the width-map section.
int64_t wmap_offset(const Geometry& g, int64_t t, int64_t k) {
  int64_t per_tile = 0, before = 0;
  for (int64_t kk = 0; kk < g.U; ++kk) {
    if (kk == k) before = per_tile;
    per_tile += 2 * g.unit_words(kk);
  }
  return t * per_tile + before;
}

inline uint16_t to_fp16_bits(double v) {
  _Float16 h = (_Float16)v;  // one correctly rounded (nearest-even) conversion
  uint16_t b;
  std::memcpy(&b, &h, 2);
  return b;
}

inline double fp16_to_double(uint16_t b) {
  _Float16 h;
  std::memcpy(&h, &b, 2);
  return (double)h;
}

inline bool fp16_finite(uint16_t b) { return (b & 0x7C00u) != 0x7C00u; }

inline uint64_t load8(const uint8_t* p) {
  uint64_t v;
  std::memcpy(&v, p, 8);
  return v;
}

// Encode 64 offset codes of width b (2b words): pair i -> word i/(16/b),
// field i%(16/b); even weight in the low half-word, odd weight in the high.
// Each step halves the distance between the codes of one half-word.
inline void encode_record(const uint8_t* u, int b, uint8_t* dst) {
  uint32_t words[16];
  if (b == 8) {
    for (int w = 0; w < 16; ++w) {
      const uint8_t* p = u + 4 * w;
      words[w] = (uint32_t)p[0] | (uint32_t)p[2] << 8 | (uint32_t)p[1] << 16 | (uint32_t)p[3] << 24;
    }
  } else if (b == 4) {
    for (int w = 0; w < 8; ++w) {
      const uint64_t x = load8(u + 8 * w);
      uint32_t half[2];
      for (int odd = 0; odd < 2; ++odd) {
        uint64_t e = (x >> (8 * odd)) & 0x000F000F000F000Full;  // four codes, 16 bits apart
        e = (e | e >> 12) & 0x000000FF000000FFull;
        half[odd] = (uint32_t)(e | e >> 24) & 0xFFFFu;
      }
      words[w] = half[0] | half[1] << 16;
    }
  } else {  // b == 2 (1-bit groups go through encode_signs)
    for (int w = 0; w < 4; ++w) {
      uint32_t half[2] = {0, 0};
      for (int k = 0; k < 2; ++k) {
        const uint64_t x = load8(u + 16 * w + 8 * k);
        for (int odd = 0; odd < 2; ++odd) {
          uint64_t e = (x >> (8 * odd)) & 0x0003000300030003ull;
          e = (e | e >> 14) & 0x0000000F0000000Full;
          half[odd] |= ((uint32_t)(e | e >> 28) & 0xFFu) << (8 * k);
        }
      }
      words[w] = half[0] | half[1] << 16;
    }
  }
  std::memcpy(dst, words, (size_t)8 * b);
}

// The 1-bit record of 64 code bits (bit i: weight i): per 32 weights the even
// bits, then the odd ones.
inline void encode_signs(uint64_t bits, uint8_t* dst) {
  uint32_t words[2];
  for (int w = 0; w < 2; ++w) {
    uint32_t x = (uint32_t)(bits >> (32 * w)), t;  // swap ever larger middle parts
    t = (x ^ (x >> 1)) & 0x22222222u;
    x ^= t ^ (t << 1);
    t = (x ^ (x >> 2)) & 0x0C0C0C0Cu;
    x ^= t ^ (t << 2);
    t = (x ^ (x >> 4)) & 0x00F000F0u;
    x ^= t ^ (t << 4);
    t = (x ^ (x >> 8)) & 0x0000FF00u;
    x ^= t ^ (t << 8);
    words[w] = x;
  }
  std::memcpy(dst, words, 8);
}

// Bit i: w[i] >= 0 (sign(0) = +1, also for -0.0).
inline uint64_t sign_bits(const float* w) {
  uint64_t m = 0;
  for (int i = 0; i < kGroup; ++i) m |= (uint64_t)(w[i] >= 0.0f) << i;
  return m;
}
// Codes clip(round(w / s), -m, m) + off, round half to even, in double.
inline void round_codes(const float* w, double s, double m, int off, uint8_t* u) {
  for (int i = 0; i < kGroup; ++i) {
    const double q = std::nearbyint((double)w[i] / s);
    u[i] = (uint8_t)((int)std::min<double>(std::max<double>(q, -m), m) + off);
  }
}

// The largest magnitude's bits; ordered as unsigned integers, NaN and Inf are
// above every finite value.
inline uint32_t top_bits(const float* w) {
  uint32_t top = 0;
  for (int i = 0; i < kGroup; ++i) {
    uint32_t v;
    std::memcpy(&v, w + i, 4);
    top = std::max(top, v & 0x7FFFFFFFu);
  }
  return top;
}
constexpr uint32_t kInfBits = 0x7F800000u;

// The 1-bit means are sums of 64 magnitudes one after the other (a chain of
// dependent additions), so up to eight groups wait here and are summed side by
// side.
constexpr int kMeans = 8;
struct MeanQueue {
  int n = 0;
  const float* w[kMeans];
  uint16_t* scale[kMeans];
};
inline void sum_magnitudes(const float* const* w, int n, double* sum) {
  for (int k = 0; k < n; ++k) {
    sum[k] = 0.0;
    for (int i = 0; i < kGroup; ++i) sum[k] += std::fabs((double)w[k][i]);
  }
}

#if defined(VBQ_PACK_AVX2)
#define VBQ_AVX2 __attribute__((target("avx2")))
VBQ_AVX2 uint64_t sign_bits_avx2(const float* w) {
  uint64_t m = 0;
  for (int i = 0; i < kGroup; i += 8) {
    const __m256 ge = _mm256_cmp_ps(_mm256_loadu_ps(w + i), _mm256_setzero_ps(), _CMP_GE_OQ);
    m |= (uint64_t)(uint32_t)_mm256_movemask_ps(ge) << i;
  }
  return m;
}
VBQ_AVX2 uint32_t top_bits_avx2(const float* w) {
  const __m256i abs = _mm256_set1_epi32(0x7FFFFFFF);
  __m256i t0 = _mm256_setzero_si256(), t1 = t0;
  for (int i = 0; i < kGroup; i += 16) {
    t0 = _mm256_max_epu32(t0, _mm256_and_si256(_mm256_loadu_si256((const __m256i*)(w + i)), abs));
    t1 = _mm256_max_epu32(t1, _mm256_and_si256(_mm256_loadu_si256((const __m256i*)(w + i + 8)), abs));
  }
  t0 = _mm256_max_epu32(t0, t1);
  __m128i x = _mm_max_epu32(_mm256_castsi256_si128(t0), _mm256_extracti128_si256(t0, 1));
  x = _mm_max_epu32(x, _mm_shuffle_epi32(x, 0x4E));
  x = _mm_max_epu32(x, _mm_shuffle_epi32(x, 0xB1));
  return (uint32_t)_mm_cvtsi128_si32(x);
}
VBQ_AVX2 void round_codes_avx2(const float* w, double s, double m, int off, uint8_t* u) {
  const __m256d sv = _mm256_set1_pd(s), hi = _mm256_set1_pd(m), lo = _mm256_set1_pd(-m);
  const __m128i ov = _mm_set1_epi32(off);
  for (int i = 0; i < kGroup; i += 16) {
    __m128i q[4];
    for (int k = 0; k < 4; ++k) {
      const __m256d x = _mm256_cvtps_pd(_mm_loadu_ps(w + i + 4 * k));
      const __m256d r = _mm256_round_pd(_mm256_div_pd(x, sv), _MM_FROUND_CUR_DIRECTION | _MM_FROUND_NO_EXC);
      q[k] = _mm_add_epi32(_mm256_cvttpd_epi32(_mm256_min_pd(_mm256_max_pd(r, lo), hi)), ov);
    }
    // codes are 1 .. 255
    _mm_storeu_si128((__m128i*)(u + i), _mm_packus_epi16(_mm_packus_epi32(q[0], q[1]), _mm_packus_epi32(q[2], q[3])));
  }
}
// Eight groups: lane k of two vectors holds group k's running sum, and every
// addition is that group's next one in order.
VBQ_AVX2 void sum_magnitudes_avx2(const float* const* w, double* sum) {
  const __m128 abs = _mm_castsi128_ps(_mm_set1_epi32(0x7FFFFFFF));
  __m256d acc[2] = {_mm256_setzero_pd(), _mm256_setzero_pd()};
  for (int i = 0; i < kGroup; i += 4) {
    for (int h = 0; h < 2; ++h) {
      __m128 a = _mm_and_ps(_mm_loadu_ps(w[4 * h] + i), abs), b = _mm_and_ps(_mm_loadu_ps(w[4 * h + 1] + i), abs);
      __m128 c = _mm_and_ps(_mm_loadu_ps(w[4 * h + 2] + i), abs), d = _mm_and_ps(_mm_loadu_ps(w[4 * h + 3] + i), abs);
      _MM_TRANSPOSE4_PS(a, b, c, d);
      acc[h] = _mm256_add_pd(acc[h], _mm256_cvtps_pd(a));
      acc[h] = _mm256_add_pd(acc[h], _mm256_cvtps_pd(b));
      acc[h] = _mm256_add_pd(acc[h], _mm256_cvtps_pd(c));
      acc[h] = _mm256_add_pd(acc[h], _mm256_cvtps_pd(d));
    }
  }
  _mm256_storeu_pd(sum, acc[0]);
  _mm256_storeu_pd(sum + 4, acc[1]);
}
// Words (u0, u2, u1, u3) of eight-bit codes.
VBQ_AVX2 void encode_bytes_avx2(const uint8_t* u, uint8_t* dst) {
  const __m256i order = _mm256_setr_epi8(0, 2, 1, 3, 4, 6, 5, 7, 8, 10, 9, 11, 12, 14, 13, 15, 0, 2, 1, 3, 4, 6, 5, 7, 8, 10,
                                         9, 11, 12, 14, 13, 15);
  for (int i = 0; i < kGroup; i += 32)
    _mm256_storeu_si256((__m256i*)(dst + i), _mm256_shuffle_epi8(_mm256_loadu_si256((const __m256i*)(u + i)), order));
}
const bool kAvx2 = __builtin_cpu_supports("avx2");
#else
constexpr bool kAvx2 = false;
inline uint64_t sign_bits_avx2(const float* w) { return sign_bits(w); }
inline uint32_t top_bits_avx2(const float* w) { return top_bits(w); }
inline void round_codes_avx2(const float* w, double s, double m, int off, uint8_t* u) { round_codes(w, s, m, off, u); }
inline void sum_magnitudes_avx2(const float* const* w, double* sum) { sum_magnitudes(w, kMeans, sum); }
inline void encode_bytes_avx2(const uint8_t* u, uint8_t* dst) { encode_record(u, 8, dst); }
#endif

// Scales of the queued 1-bit groups.
inline vbq_status flush_means(MeanQueue* mq) {
  double sum[kMeans];
  if (kAvx2 && mq->n == kMeans)
    sum_magnitudes_avx2(mq->w, sum);
  else
    sum_magnitudes(mq->w, mq->n, sum);
  vbq_status st = VBQ_OK;
  for (int k = 0; k < mq->n; ++k) {
    *mq->scale[k] = to_fp16_bits(sum[k] / kGroup);
    if (!fp16_finite(*mq->scale[k])) st = VBQ_ERR_SCALE_RANGE;
  }
  mq->n = 0;
  return st;
}

// Quantize one group (paper section 3.1) and write its record and fp16 scale
// (a 1-bit group's scale when the queue is flushed).
inline vbq_status quantize_group(const float* w, int b, uint8_t* dst, uint16_t* s_bits, MeanQueue* mq) {
  const uint32_t top = kAvx2 ? top_bits_avx2(w) : top_bits(w);
  if (top >= kInfBits) return VBQ_ERR_NONFINITE;
  if (b == 1) {
    encode_signs(kAvx2 ? sign_bits_avx2(w) : sign_bits(w), dst);
    mq->w[mq->n] = w;
    mq->scale[mq->n] = s_bits;
    return ++mq->n == kMeans ? flush_means(mq) : VBQ_OK;
  }
  const int m = (1 << (b - 1)) - 1;
  float amax;
  std::memcpy(&amax, &top, 4);
  uint16_t sb = to_fp16_bits((double)amax / m);
  if (!fp16_finite(sb)) return VBQ_ERR_SCALE_RANGE;
  *s_bits = sb;
  const double s = fp16_to_double(sb);  // codes use the stored scale
  const int off = 1 << (b - 1);
  uint8_t u[kGroup];
  if (s == 0.0)
    std::memset(u, off, sizeof(u));
  else if (kAvx2)
    round_codes_avx2(w, s, m, off, u);
  else
    round_codes(w, s, m, off, u);
  if (kAvx2 && b == 8)
    encode_bytes_avx2(u, dst);
  else
    encode_record(u, b, dst);
  return VBQ_OK;
}

// The record of already-quantized levels, with level-set validation.
inline vbq_status record_of_levels(const int8_t* q, int b, uint8_t* dst) {
  if (b == 1) {
    uint64_t m = 0;
    bool ok = true;
    for (int i = 0; i < kGroup; ++i) {
      ok &= (q[i] == 1) | (q[i] == -1);
      m |= (uint64_t)(q[i] > 0) << i;
    }
    if (!ok) return VBQ_ERR_CODE_RANGE;
    encode_signs(m, dst);
    return VBQ_OK;
  }
  const int m = (1 << (b - 1)) - 1, off = 1 << (b - 1);
  uint8_t u[kGroup];
  int lo = 0, hi = 0;
  for (int i = 0; i < kGroup; ++i) {
    lo = std::min<int>(lo, q[i]);
    hi = std::max<int>(hi, q[i]);
    u[i] = (uint8_t)(q[i] + off);
  }
  if (lo < -m || hi > m) return VBQ_ERR_CODE_RANGE;
  encode_record(u, b, dst);
  return VBQ_OK;
}

struct Source {
  const float* W = nullptr;         // vbq_pack
  const int8_t* q = nullptr;        // vbq_pack_codes
  const uint16_t* scales = nullptr;  // vbq_pack_codes
};

// Quantize or encode group (r, j): its record, and its fp16 scale (a quantized
// 1-bit group's when the queue is flushed).
inline vbq_status pack_group(const Geometry& g, const Source& src, int64_t r, int64_t j, int b, uint8_t* dst,
                             uint16_t* scale, MeanQueue* mq) {
  if (src.W) return quantize_group(src.W + r * g.K + j * kGroup, b, dst, scale, mq);
  const vbq_status st = record_of_levels(src.q + r * g.K + j * kGroup, b, dst);
  if (st != VBQ_OK) return st;
  const uint16_t sb = src.scales[r * g.G + j];
  if (!fp16_finite(sb)) return VBQ_ERR_NONFINITE;
  if (sb & 0x8000u) return VBQ_ERR_SCALE_RANGE;
  *scale = sb;
  return VBQ_OK;
}

// The status of tile t's first refused group in the order of the entries (down
// each column), which is the one reported; the packing itself goes by rows and
// knows a 1-bit mean only later.
__attribute__((cold)) vbq_status first_refused(const Geometry& g, const Source& src, const uint8_t* bits, int64_t t) {
  uint8_t record[8 * 8];
  uint16_t scale;
  MeanQueue mq;
  for (int64_t j = 0; j < g.G; ++j) {
    for (int64_t rl = 0; rl < g.tile_rows(t); ++rl) {
      const int64_t r = t * g.R + rl;
      vbq_status st = pack_group(g, src, r, j, bits[r * g.G + j], record, &scale, &mq);
      if (st == VBQ_OK) st = flush_means(&mq);
      if (st != VBQ_OK) return st;
    }
  }
  return VBQ_OK;
}

vbq_status pack_impl(int64_t N, int64_t K, const Source& src, const uint8_t* bits,
                     const vbq_pack_opts* opts, void* blob, size_t blob_bytes, vbq_desc* desc) {
  if (!bits || !blob || !desc) return VBQ_ERR_NULL;
  Geometry g;
  vbq_status st = make_geometry(N, K, opts, &g);
  if (st != VBQ_OK) return st;
  if (opts && opts->flags != 0) return VBQ_ERR_UNSUPPORTED;
  if ((uintptr_t)blob % 8 != 0) return VBQ_ERR_BUFFER;
  const uint32_t n_threads = opts ? opts->n_threads : 0;
  Counts cnt;
  if ((st = count_units(g, bits, n_threads, &cnt)) != VBQ_OK) return st;
  std::vector<uint32_t> starts;
  int64_t n_entries[4];
  if ((st = unit_starts(g, cnt, &starts, n_entries)) != VBQ_OK) return st;
  vbq_desc d;
  fill_desc_header(g, n_entries, &d);
  if (blob_bytes < d.total_bytes) return VBQ_ERR_BUFFER;

  uint8_t* base = (uint8_t*)blob;
  // zero the alignment padding between sections and after the last one
  uint64_t pos = 0;
  for (int s = 0; s < VBQ_NSECTIONS; ++s) {
    if (d.section_off[s] > pos) std::memset(base + pos, 0, d.section_off[s] - pos);
    pos = std::max<uint64_t>(pos, d.section_off[s] + d.section_len[s]);
  }
  if (d.total_bytes > pos) std::memset(base + pos, 0, d.total_bytes - pos);

  uint32_t* units = (uint32_t*)(base + d.section_off[VBQ_SEC_UNITS]);
  uint64_t* wmap = (uint64_t*)(base + d.section_off[VBQ_SEC_WMAP]);
  uint8_t* codes[4];
  uint16_t* scales[4];
  for (int c = 0; c < 4; ++c) {
    codes[c] = base + d.section_off[VBQ_SEC_CODES0 + c];
    scales[c] = (uint16_t*)(base + d.section_off[VBQ_SEC_SCALES0 + c]);
  }
  // unit table, including the totals row
  for (int64_t u = 0; u <= g.units; ++u) {
    uint32_t* row = units + (size_t)u * kUnitRowWords;
    for (int c = 0; c < 4; ++c) row[c] = starts[(size_t)u * 4 + c];
    row[4] = (uint32_t)(u < g.units ? wmap_offset(g, u / g.U, u % g.U) : g.wmap_words);
    row[5] = row[6] = row[7] = 0;
  }

  std::atomic<int> err{VBQ_OK};
  parallel_tiles(g.T, n_threads, g.N * g.G, kPackGrain, [&](int64_t t) {
    if (err.load(std::memory_order_relaxed) != VBQ_OK) return;
    const int64_t rows = g.tile_rows(t);
    std::vector<uint64_t> planes;
    std::vector<uint32_t> entry;  // of each position of the unit, rows together
    MeanQueue mq;
    for (int64_t k = 0; k < g.U; ++k) {
      const int64_t unit = t * g.U + k;
      const int64_t W = g.unit_words(k), cols = g.chunk_cols(k), j0 = k * g.C;
      planes.assign((size_t)2 * W, 0);
      entry.resize((size_t)(rows * cols));
      uint32_t next[4];
      for (int c = 0; c < 4; ++c) next[c] = starts[(size_t)unit * 4 + c];
      for (int64_t jl = 0; jl < cols; ++jl) {  // entries go by position: down each column
        for (int64_t rl = 0; rl < rows; ++rl) {
          const int64_t p = jl * g.R + rl;
          const uint64_t c = (uint64_t)class_of_bits(bits[(t * g.R + rl) * g.G + j0 + jl]);
          planes[(size_t)(p >> 6)] |= (c & 1) << (p & 63);
          planes[(size_t)(W + (p >> 6))] |= (c >> 1) << (p & 63);
          entry[(size_t)(rl * cols + jl)] = next[c]++;
        }
      }
      for (int64_t rl = 0; rl < rows; ++rl) {  // the weights go by row, as they lie in memory
        const int64_t r = t * g.R + rl;
        for (int64_t jl = 0; jl < cols; ++jl) {
          const int64_t j = j0 + jl;
          const int b = bits[r * g.G + j];
          const int c = class_of_bits((uint8_t)b);
          const uint32_t e = entry[(size_t)(rl * cols + jl)];
          if (pack_group(g, src, r, j, b, codes[c] + (size_t)e * (8u << c), &scales[c][e], &mq) != VBQ_OK) {
            record_error(err, first_refused(g, src, bits, t));
            return;
          }
        }
      }
      std::memcpy(wmap + units[(size_t)unit * kUnitRowWords + 4], planes.data(), planes.size() * 8);
    }
    if (flush_means(&mq) != VBQ_OK) record_error(err, first_refused(g, src, bits, t));
  });
  if (err.load() != VBQ_OK) return (vbq_status)err.load();
  *desc = d;
  return VBQ_OK;
}

}  // namespace

extern "C" {

const char* vbq_status_string(vbq_status s) {
  switch (s) {
    case VBQ_OK: return "ok";
    case VBQ_ERR_NULL: return "null pointer";
    case VBQ_ERR_SHAPE: return "unsupported shape (need N >= 1, K >= 64, K % 64 == 0; 0 <= M <= 16)";
    case VBQ_ERR_BITS: return "bit-width outside {1,2,4,8}";
    case VBQ_ERR_CODE_RANGE: return "level outside the level set of its width";
    case VBQ_ERR_NONFINITE: return "non-finite weight or scale";
    case VBQ_ERR_SCALE_RANGE: return "scale overflows fp16 or is negative";
    case VBQ_ERR_BUFFER: return "buffer too small or misaligned";
    case VBQ_ERR_DESC: return "descriptor does not match this layout";
    case VBQ_ERR_HIP: return "HIP runtime error";
    case VBQ_ERR_UNSUPPORTED: return "unsupported option";
  }
  return "unknown status";
}

uint32_t vbq_layout_version(void) { return VBQ_LAYOUT_VERSION; }

vbq_status vbq_pack_size(int64_t N, int64_t K, const uint8_t* bits, const vbq_pack_opts* opts,
                         size_t* bytes, vbq_desc* desc_out) {
  if (!bits || !bytes) return VBQ_ERR_NULL;
  Geometry g;
  vbq_status st = make_geometry(N, K, opts, &g);
  if (st != VBQ_OK) return st;
  if (opts && opts->flags != 0) return VBQ_ERR_UNSUPPORTED;
  Counts cnt;
  if ((st = count_units(g, bits, opts ? opts->n_threads : 0, &cnt)) != VBQ_OK) return st;
  std::vector<uint32_t> starts;
  int64_t n_entries[4];
  if ((st = unit_starts(g, cnt, &starts, n_entries)) != VBQ_OK) return st;
  vbq_desc d;
  fill_desc_header(g, n_entries, &d);
  *bytes = (size_t)d.total_bytes;
  if (desc_out) *desc_out = d;
  return VBQ_OK;
}

vbq_status vbq_pack(int64_t N, int64_t K, const float* W, const uint8_t* bits,
                    const vbq_pack_opts* opts, void* blob, size_t blob_bytes, vbq_desc* desc) {
  if (!W) return VBQ_ERR_NULL;
  Source src;
  src.W = W;
  return pack_impl(N, K, src, bits, opts, blob, blob_bytes, desc);
}

vbq_status vbq_pack_codes(int64_t N, int64_t K, const int8_t* q, const uint16_t* scale_f16,
                          const uint8_t* bits, const vbq_pack_opts* opts, void* blob,
                          size_t blob_bytes, vbq_desc* desc) {
  if (!q || !scale_f16) return VBQ_ERR_NULL;
  Source src;
  src.q = q;
  src.scales = scale_f16;
  return pack_impl(N, K, src, bits, opts, blob, blob_bytes, desc);
}

namespace {

// Rows of each width in increasing row order, and the widths present.
vbq_status bucket_rows(int64_t N, const uint8_t* row_bits, std::vector<int64_t> rows[4]) {
  for (int64_t n = 0; n < N; ++n) {
    const int c = class_of_bits(row_bits[n]);
    if (c < 0) return VBQ_ERR_BITS;
    rows[c].push_back(n);
  }
  return VBQ_OK;
}

// Descriptor and byte size of one bucket (n rows of width 2^c, K columns).
vbq_status bucket_desc(int64_t n, int64_t K, int c, const vbq_pack_opts* opts, vbq_desc* d) {
  Geometry g;
  vbq_status st = make_geometry(n, K, opts, &g);
  if (st != VBQ_OK) return st;
  int64_t n_entries[4] = {0, 0, 0, 0};
  n_entries[c] = n * g.G;
  if (n_entries[c] > 0xFFFFFFFFll || g.wmap_words > 0xFFFFFFFFll) return VBQ_ERR_UNSUPPORTED;
  fill_desc_header(g, n_entries, d);
  return VBQ_OK;
}

}  // namespace

vbq_status vbq_pack_row_buckets_size(int64_t N, int64_t K, const uint8_t* row_bits, const vbq_pack_opts* opts,
                                     size_t* bytes, int32_t* n_buckets) {
  if (!row_bits || !bytes || !n_buckets) return VBQ_ERR_NULL;
  if (N < 1 || K < kGroup || K % kGroup != 0) return VBQ_ERR_SHAPE;
  if (opts && opts->flags != 0) return VBQ_ERR_UNSUPPORTED;
  std::vector<int64_t> rows[4];
  vbq_status st = bucket_rows(N, row_bits, rows);
  if (st != VBQ_OK) return st;
  uint64_t total = 0;
  int32_t nb = 0;
  for (int c = 0; c < 4; ++c) {
    if (rows[c].empty()) continue;
    vbq_desc d;
    if ((st = bucket_desc((int64_t)rows[c].size(), K, c, opts, &d)) != VBQ_OK) return st;
    total = align_up(total) + d.total_bytes;
    ++nb;
  }
  *bytes = (size_t)total;
  *n_buckets = nb;
  return VBQ_OK;
}

vbq_status vbq_pack_row_buckets(int64_t N, int64_t K, const int8_t* q, const uint16_t* scale_f16,
                                const uint8_t* row_bits, const vbq_pack_opts* opts, void* blob, size_t blob_bytes,
                                vbq_bucket buckets[VBQ_MAX_BUCKETS], int32_t* n_buckets, int32_t* row_index) {
  if (!q || !scale_f16 || !row_bits || !blob || !buckets || !n_buckets || !row_index) return VBQ_ERR_NULL;
  size_t need = 0;
  int32_t nb = 0;
  vbq_status st = vbq_pack_row_buckets_size(N, K, row_bits, opts, &need, &nb);
  if (st != VBQ_OK) return st;
  if ((uintptr_t)blob % 8 != 0 || blob_bytes < need) return VBQ_ERR_BUFFER;
  std::vector<int64_t> rows[4];
  bucket_rows(N, row_bits, rows);
  const int64_t G = K / kGroup;
  uint64_t off = 0;
  int64_t row_begin = 0;
  int32_t i = 0;
  std::vector<int8_t> qb;
  std::vector<uint16_t> sb;
  std::vector<uint8_t> bb;
  for (int c = 0; c < 4; ++c) {
    const int64_t n = (int64_t)rows[c].size();
    if (n == 0) continue;
    // the bucket's rows, gathered in order: the same input vbq_pack_codes
    // would get for these rows alone
    qb.resize((size_t)(n * K));
    sb.resize((size_t)(n * G));
    bb.assign((size_t)(n * G), (uint8_t)(1u << c));
    for (int64_t r = 0; r < n; ++r) {
      const int64_t src = rows[c][(size_t)r];
      std::memcpy(&qb[(size_t)(r * K)], q + src * K, (size_t)K);
      std::memcpy(&sb[(size_t)(r * G)], scale_f16 + src * G, (size_t)G * 2);
      row_index[row_begin + r] = (int32_t)src;
    }
    off = align_up(off);
    vbq_bucket& b = buckets[i];
    b = vbq_bucket{};
    b.bits = 1 << c;
    b.row_begin = row_begin;
    b.n_rows = n;
    b.blob_offset = off;
    Source src;
    src.q = qb.data();
    src.scales = sb.data();
    st = pack_impl(n, K, src, bb.data(), opts, (uint8_t*)blob + off, blob_bytes - off, &b.desc);
    if (st != VBQ_OK) return st;
    off += b.desc.total_bytes;
    row_begin += n;
    ++i;
  }
  *n_buckets = nb;
  return VBQ_OK;
}

vbq_status vbq_desc_check(const vbq_desc* d) {
  if (!d) return VBQ_ERR_NULL;
  if (d->magic != VBQ_MAGIC || d->version != VBQ_LAYOUT_VERSION || d->group != kGroup) return VBQ_ERR_DESC;
  vbq_pack_opts o{d->tile_rows, d->chunk_groups, 0, 0};
  Geometry g;
  if (make_geometry(d->N, d->K, &o, &g) != VBQ_OK) return VBQ_ERR_DESC;
  if (g.T != d->n_tiles || g.U != d->n_chunks || g.units != d->n_units) return VBQ_ERR_DESC;
  int64_t total = 0;
  for (int c = 0; c < 4; ++c) {
    if (d->n_entries[c] < 0) return VBQ_ERR_DESC;
    total += d->n_entries[c];
  }
  if (total != g.N * g.G) return VBQ_ERR_DESC;
  vbq_desc ref;
  fill_desc_header(g, d->n_entries, &ref);
  for (int s = 0; s < VBQ_NSECTIONS; ++s)
    if (ref.section_off[s] != d->section_off[s] || ref.section_len[s] != d->section_len[s]) return VBQ_ERR_DESC;
  if (ref.total_bytes != d->total_bytes) return VBQ_ERR_DESC;
  return VBQ_OK;
}

}  // extern "C"
