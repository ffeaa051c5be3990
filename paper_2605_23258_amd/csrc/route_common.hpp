// What the routing kernels share: order-preserving keys, bucket maps, scans, the pooling of the attention
// mass, and the description of the packed cache's row copies.
#pragma once
#include "common.hpp"
#include "launch.hpp"

namespace vec {

namespace {

// Order-preserving map float -> u32 (larger float, larger key); -0 and +0 share a key.
__device__ __forceinline__ uint32_t float_key(float x) {
  uint32_t b = __float_as_uint(x + 0.0f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Leading digit of a key: which of the 2048 buckets of the first radix level it falls in.  Plain:
// the key's top 11 bits, a quarter of an octave of scores per bucket.  When the scorer has told
// where the bulk of a head's scores lies, 2046 buckets of 2^shift keys each are laid over that
// range instead, so that scores which agree in their leading bits (a flat attention row: every
// score within a few per cent of 1/n) still spread over the buckets; bucket 0 takes every key below
// the range and bucket 2047 every key above it (attention sinks, the +inf of the window columns).
// Keys of one bucket between 1 and 2046 agree in all bits from `shift` up; the two end buckets
// (and they alone) may hold keys that differ anywhere.  Wherever a score falls the select stays
// exact: the range only decides how evenly the buckets fill.
struct DigitMap {
  uint32_t lowq;
  int shift;
  __device__ __forceinline__ bool plain() const { return shift == 21 && lowq == 0u; }
  __device__ __forceinline__ uint32_t digit(uint32_t key) const {
    // a saturating difference: written with max (a compare-and-select around `q - lowq` is folded away by
    // this compiler at -O3, which then lets the difference wrap)
    const uint32_t q = key >> shift;
    return min(max(q, lowq) - lowq, 2047u);
  }
};
// 2046 buckets of 2^shift keys each over [klo, khi], shift as small as that allows
__device__ __forceinline__ DigitMap digit_map_for_keys(uint32_t klo, uint32_t khi) {
  DigitMap plain = {0u, 21};
  if (khi < klo) return plain;
  // (khi >> s) - (klo >> s) <= ((khi - klo) >> s) + 1: start where the difference has 11 bits left
  const uint32_t diff = khi - klo;
  int s = diff ? max(0, 21 - (int)__clz(diff)) : 0;
  if ((khi >> s) - (klo >> s) > 2045u) ++s;
  if (s >= 21) return plain;
  DigitMap m = {max(klo >> s, 1u) - 1u, s};
  return m;
}
// cnt, sum_l, sum_ll: over the head's prefix columns of positive attention mass m, their number and
// the sums of l = log2(m) - log_ref and of l * l.  The buckets cover the mean of log2(m) give or
// take four standard deviations (and a 64th of an octave, so that equal masses still get a
// range): at most a sixteenth of the columns lie outside, whatever their distribution, and a few
// columns far from the rest (attention sinks, the zero-padded edges of the pooling) move the range
// very little.
__device__ __forceinline__ DigitMap digit_map_for_stats(float cnt, float sum_l, float sum_ll, float log_ref) {
  DigitMap plain = {0u, 21};
  if (!(cnt >= 1.f)) return plain;
  // hardware reciprocal, square root and exponential: a rough range is all that is needed, and
  // every wave of the head gets the same bits from the same inputs
  const float inv = __builtin_amdgcn_rcpf(cnt);
  const float mu = sum_l * inv;
  const float sd = __builtin_amdgcn_sqrtf(fmaxf(sum_ll * inv - mu * mu, 0.f));
  const float mid = log_ref + mu, half = 4.f * sd + 0.015625f;
  if (!(mid - half > -120.f) || !(mid + half < 120.f)) return plain;        // also NaN
  return digit_map_for_keys(float_key(__builtin_amdgcn_exp2f(mid - half)), float_key(__builtin_amdgcn_exp2f(mid + half)));
}
// The same from a sample of the keys themselves, for scores of any sign that arrive without
// statistics (vector_route on its own): cnt keys k = key >> 12 with sum s1 and sum of squares s2.
// For positive floats the key is linear in the score inside an octave and counts octaves across
// them, so its mean and deviation bound the bulk the same way.
__device__ __forceinline__ DigitMap digit_map_for_sample(unsigned long long cnt, unsigned long long s1, unsigned long long s2) {
  DigitMap plain = {0u, 21};
  if (cnt < 32) return plain;
  const double inv = 1.0 / (double)cnt, mu = (double)s1 * inv;
  const double var = (double)s2 * inv - mu * mu;
  const double half = 4.0 * sqrt(var > 0.0 ? var : 0.0) + 32.0;             // 32 * 4096 keys: a 64th of an octave
  const double lo = (mu - half) * 4096.0, hi = (mu + half) * 4096.0;
  const uint32_t klo = lo > 0.0 ? (uint32_t)lo : 0u, khi = hi < 4294967295.0 ? (uint32_t)hi : 0xffffffffu;
  return digit_map_for_keys(klo, khi);
}

// ---------------------------------------------------------------------------
// prefix sums inside a wave on the DPP network
// ---------------------------------------------------------------------------
__device__ __forceinline__ int wave_total_of_scan(int incl) { return __builtin_amdgcn_readlane(incl, 63); }


// Average pooling ends in sum / kernel, correctly rounded with three instructions instead of a division's ten: the
// product with the rounded reciprocal, corrected once by the remainder (P. Markstein, IBM J. Res. Dev. 34 (1990),
// 111-119).  Why that is enough here: kernel is an odd integer, below 2^21 say.  The remainder sum - q * kernel is then a
// whole number, below 2^24, of q's last places, so the inner fma is exact, also for denormals.  And sum / kernel
// lies at least 1 / (4 kernel) of a last place away from the middle between two floats, further than the
// reciprocal's error in the correction (2^-23 of a last place) can move it.
__device__ __forceinline__ float pool_mean(float sum, float kernel, float inv_kernel) {
  const float q = sum * inv_kernel;
  return fmaf(fmaf(-q, kernel, sum), inv_kernel, q);
}

struct GatherParams {
  const unsigned char* k; const unsigned char* v;
  int64_t k_sh, k_st, v_sh, v_st;          // byte strides
  int hps;                                 // stacked sequences: KV heads per sequence (0: one sequence)
  int64_t k_sb, v_sb;                      // byte strides between sequences
  const int32_t* idx_retain; const int32_t* idx_approx;
  int n_retain, n_approx, cap_retain, row_bytes, n;
  unsigned char* k_ret; unsigned char* v_ret; unsigned char* k_apx;
};

inline GatherParams gather_params(const vector_shape& s, const void* k, const void* v, const int32_t* idx_retain, const int32_t* idx_approx,
                           int n_retain, int n_approx, void* k_ret, void* v_ret, void* k_apx, int cap_retain, const SeqStack* stack) {
  const int esz = (s.dtype == VECTOR_BF16) ? 2 : 4;
  GatherParams p;
  p.k = reinterpret_cast<const unsigned char*>(k);
  p.v = reinterpret_cast<const unsigned char*>(v);
  const int64_t k_st = s.k_stride_tok ? s.k_stride_tok : s.head_dim;
  const int64_t v_st = s.v_stride_tok ? s.v_stride_tok : s.head_dim;
  p.k_st = k_st * esz;
  p.v_st = v_st * esz;
  p.k_sh = (s.k_stride_head ? s.k_stride_head : (int64_t)s.seq_len * k_st) * esz;
  p.v_sh = (s.v_stride_head ? s.v_stride_head : (int64_t)s.seq_len * v_st) * esz;
  p.hps = stack ? stack->heads_per_seq : 0;
  p.k_sb = stack ? stack->k_stride_seq * esz : 0;
  p.v_sb = stack ? stack->v_stride_seq * esz : 0;
  p.idx_retain = idx_retain; p.idx_approx = idx_approx;
  p.n_retain = n_retain; p.n_approx = n_approx; p.cap_retain = cap_retain;
  p.row_bytes = s.head_dim * esz; p.n = s.seq_len;
  p.k_ret = reinterpret_cast<unsigned char*>(k_ret);
  p.v_ret = reinterpret_cast<unsigned char*>(v_ret);
  p.k_apx = reinterpret_cast<unsigned char*>(k_apx);
  return p;
}

// ---------------------------------------------------------------------------
// workgroups of NT threads (512 or 1024): scans, histogram picks, emission and row copies
// ---------------------------------------------------------------------------
template <int NT> constexpr int kWaves = NT / kWave;
template <int NT> constexpr int kBlock = NT * 4;        // tokens per block: four consecutive ones per thread
constexpr int kHeadBins = 2048;
constexpr int kRankCap = 256;                   // candidates ranked by comparison

typedef __attribute__((ext_vector_type(4), aligned(4))) uint32_t u32x4_u;

// Workgroup barrier for data in LDS alone: global loads in flight (the residuals, while the scores are worked
// on) and stores (score, tiers, lists) are not waited for.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// packed pairs of counts: retained in the low half, approximated in the high one
__device__ __forceinline__ int low16(int x) { return x & 0xffff; }
__device__ __forceinline__ int high16(int x) { return (int)((uint32_t)x >> 16); }

// sum of a float over the waves' entries, the same bits in every lane
template <int NT> __device__ __forceinline__ float sum_of_waves(const float* row, int lane) {
  static_assert(kWaves<NT> == 8 || kWaves<NT> == 16, "a row of lanes");
  float x = row[lane & (kWaves<NT> - 1)];
  x += dpp_take_f<0x111, 0xf>(0.f, x);
  x += dpp_take_f<0x112, 0xf>(0.f, x);
  x += dpp_take_f<0x114, 0xf>(0.f, x);
  if constexpr (kWaves<NT> == 16) x += dpp_take_f<0x118, 0xf>(0.f, x);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), kWaves<NT> - 1));
}

// inclusive prefix over the waves' entries, one per lane
template <int NT> __device__ __forceinline__ int row_incl_scan(int x) {
  x += dpp_take<0x111, 0xf>(x);
  x += dpp_take<0x112, 0xf>(x);
  x += dpp_take<0x114, 0xf>(x);
  if constexpr (kWaves<NT> == 16) x += dpp_take<0x118, 0xf>(x);
  return x;
}

// exclusive prefix over the workgroup's threads of a packed pair of counts, and the total; row: [waves]
template <int NT> __device__ __forceinline__ void head_scan(int v, int* row, int& before, int& total) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int incl = wave_incl_scan_dpp(v);
  if (lane == 63) row[wave] = incl;
  lds_barrier();
  const int x = row_incl_scan<NT>(row[lane & (kWaves<NT> - 1)]);          // every lane one wave's total
  const int upto = wave ? __builtin_amdgcn_readlane(x, wave - 1) : 0;
  total = __builtin_amdgcn_readlane(x, kWaves<NT> - 1);
  before = upto + incl - v;
}

template <int NT> __device__ __forceinline__ void clear_bins(int* hist) {
  if constexpr (kHeadBins == 4 * NT) *reinterpret_cast<int4*>(hist + 4 * threadIdx.x) = make_int4(0, 0, 0, 0);
  else {
    static_assert(kHeadBins == 2 * NT, "two or four buckets per thread");
    *reinterpret_cast<int2*>(hist + 2 * threadIdx.x) = make_int2(0, 0);
  }
}

// histogram counts -> the bucket with #(keys above it) < k <= #(keys in or above it); row: [waves], pick: [3]
template <int NT> __device__ __forceinline__ void pick_bin(const int* hist, int* row, int* pick, int k, int& d, int& above, int& count) {
  constexpr int BPT = kHeadBins / NT;
  const int lo = kHeadBins - BPT - BPT * (int)threadIdx.x;
  int c[BPT], sum = 0;                           // buckets lo ..
#pragma unroll
  for (int q = 0; q < BPT; ++q) { c[q] = hist[lo + q]; sum += c[q]; }
  int before, total;
  head_scan<NT>(sum, row, before, total);
  if (before < k && k <= before + sum) {
    int b = lo + BPT - 1, in = c[BPT - 1];
#pragma unroll
    for (int q = BPT - 2; q >= 0; --q)
      if (b == lo + q + 1 && k > before + in) { before += in; in = c[q]; --b; }
    pick[0] = b; pick[1] = before; pick[2] = in;
  }
  lds_barrier();
  d = __builtin_amdgcn_readfirstlane(pick[0]); above = __builtin_amdgcn_readfirstlane(pick[1]); count = __builtin_amdgcn_readfirstlane(pick[2]);
}

// A sample's count, sum and sum of squares (in units of 4096 keys about the center) -> where to lay the buckets
__device__ __forceinline__ DigitMap digit_map_about(uint32_t center, float cnt, float s1, float s2) {
  DigitMap map = {0u, 21};
  if (cnt >= 32.f) {
    const float inv = __builtin_amdgcn_rcpf(cnt), mu = s1 * inv;
    const float half = 4.f * __builtin_amdgcn_sqrtf(fmaxf(s2 * inv - mu * mu, 0.f)) + 32.f;
    const float mid = (float)(center >> 12) + mu;
    map = digit_map_for_keys((uint32_t)fmaxf(mid - half, 0.f) << 12, (uint32_t)fminf(mid + half, 1048575.f) << 12);
  }
  return map;
}
// the keys of bucket d: [lo, lo + span]; no key is 0
__device__ __forceinline__ void bucket_range(const DigitMap& map, int d, uint32_t& lo, uint32_t& span) {
  if (map.plain()) {
    lo = (uint32_t)d << 21;
    span = (1u << 21) - 1u;
  } else {
    lo = d == 0 ? 0u : (map.lowq + (uint32_t)d) << map.shift;
    const uint32_t hi = d == 2047 ? 0xffffffffu : ((map.lowq + (uint32_t)d + 1u) << map.shift) - 1u;
    span = hi - lo;
  }
  if (lo == 0u) { lo = 1u; span -= 1u; }
}

// ---------------------------------------------------------------------------
// many keys in one bucket: scores that are equal or nearly so (attention rows that underflow to zero, scorers
// with few values)
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x111, 0xf, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x112, 0xf, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x114, 0xf, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x118, 0xf, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x142, 0xa, 0xf, false));
  v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x143, 0xc, 0xf, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// smallest and largest of the workgroup's keys in [lo, lo + span]; each(f) hands every key to f; row: [2][waves], free
// until the barrier after this
template <int NT, typename Each>
__device__ __forceinline__ void key_range(Each each, uint32_t lo, uint32_t span, uint32_t (*row)[kWaves<NT>], uint32_t& least, uint32_t& most) {
  uint32_t a = 0xffffffffu, b = 0u;
  each([&](uint32_t x) {
    const bool in = x - lo <= span;
    a = min(a, in ? x : 0xffffffffu);
    b = max(b, in ? x : 0u);
  });
  a = wave_min_u32(a);
  b = ~wave_min_u32(~b);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { row[0][wave] = a; row[1][wave] = b; }
  lds_barrier();
#pragma unroll
  for (int w = 0; w < kWaves<NT>; ++w) { a = min(a, row[0][w]); b = max(b, row[1][w]); }
  least = (uint32_t)__builtin_amdgcn_readfirstlane((int)a);
  most = (uint32_t)__builtin_amdgcn_readfirstlane((int)b);
}

// Of the `count` keys in [lo, lo + span] the k-th largest is wanted: cuts the range until it holds at most kRankCap
// keys, or one number (span 0).  Where the keys lie in it is looked up before they are counted: equal keys need
// no count at all, and 64 lanes that add to the same word of a histogram take 64 turns (7 us for 16384 equal
// keys, against 1 us for the look).  The buckets come in several copies, a lane's own by its number, for the same
// reason.  tight: [lo, lo + span] starts and ends with a key already.
template <int NT, typename Each>
__device__ __forceinline__ void narrow(Each each, bool tight, uint32_t& lo, uint32_t& span, int& k, int& count, int* hist, int* row, int* pick,
                                       uint32_t (*range)[kWaves<NT>]) {
  const int lane = threadIdx.x & 63;
  while (__builtin_expect(count > kRankCap && span != 0u, 0)) {         // uniform
    if (!tight) {
      uint32_t most;
      key_range<NT>(each, lo, span, range, lo, most);
      span = most - lo;
      if (span == 0u) break;
    }
    tight = false;
    const int s = max(0, 23 - (int)__clz(span));                        // at most 512 buckets over the range,
    const uint32_t last = span >> s;
    const int copies_log = min(6, (int)__clz(last) - 21);               // 4 to 64 copies of each
    const int copy = lane & ((1 << copies_log) - 1);
    clear_bins<NT>(hist);
    lds_barrier();
    each([&](uint32_t x) { if (x - lo <= span) atomicAdd(&hist[(int)(((x - lo) >> s) << copies_log) + copy], 1); });
    lds_barrier();
    int sum = 0;                                                        // a bucket's copies lie side by side
    if ((int)threadIdx.x < (kHeadBins >> copies_log))
      for (int j = 0; j < (1 << copies_log); ++j) sum += hist[((int)threadIdx.x << copies_log) + ((j + lane) & ((1 << copies_log) - 1))];
    lds_barrier();
    hist[threadIdx.x] = sum;
#pragma unroll
    for (int q = 1; q < kHeadBins / NT; ++q) hist[q * NT + threadIdx.x] = 0;
    lds_barrier();
    int d, above;
    pick_bin<NT>(hist, row, pick, k, d, above, count);
    k -= above;
    lo += (uint32_t)d << s;
    span = min(span - ((uint32_t)d << s), (1u << s) - 1u);
  }
}

// Whether the k-th largest key lies among those that agree with `center` but for their last 12 bits; then lo, span,
// k and count describe these.  Worth a try where every key of a sample does (its sum of squares about the
// center is 0): a histogram would put all of them into a few words.  row: [waves]
template <int NT, typename Each>
__device__ __forceinline__ bool around_center(Each each, uint32_t center, uint32_t& lo, uint32_t& span, int& k, int& count, int* row) {
  const uint32_t first = center & ~0xfffu;
  int in = 0, above = 0;
  each([&](uint32_t x) {
    in += x - first <= 0xfffu;
    above += x > first + 0xfffu;
  });
  int unused, total_in, total_above;
  head_scan<NT>(in, row, unused, total_in);
  lds_barrier();                                                        // the row is used again
  head_scan<NT>(above, row, unused, total_above);
  if (k <= total_above || k > total_above + total_in) return false;    // uniform
  lo = first;
  span = 0xfffu;
  k -= total_above;
  count = total_in;
  return true;
}

// Where a head's results go.
struct EmitTarget {
  uint8_t* tier; int32_t* ir; int32_t* ia;       // of the head
  int n, n_retain, n_approx;
};
// A thread's four tokens t0 .. t0 + 3 (bit e of ret4 / apx4: token t0 + e) into the workgroup's list, which holds the own_r
// retained tokens that it emits, then the approximated ones; at_r, at_a: the thread's first places among each.
__device__ __forceinline__ void list_tokens(int t0, uint32_t ret4, uint32_t apx4, int at_r, int at_a, int own_r, int* list) {
  at_a += own_r;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int r = (int)((ret4 >> e) & 1u), a = (int)((apx4 >> e) & 1u);
    if (r | a) list[r ? at_r : at_a] = t0 + e;
    at_r += r;
    at_a += a;
  }
}
__device__ __forceinline__ void store_tiers(const EmitTarget& o, int t0, uint32_t ret4, uint32_t apx4) {
  uint32_t word = 0u;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    word |= ((ret4 >> e) & 1u ? (uint32_t)VECTOR_TIER_RETAIN : (apx4 >> e) & 1u ? (uint32_t)VECTOR_TIER_APPROX : (uint32_t)VECTOR_TIER_EVICT) << (8 * e);
  if ((reinterpret_cast<uintptr_t>(o.tier) & 3u) == 0 && t0 + 4 <= o.n) {
    *reinterpret_cast<uint32_t*>(o.tier + t0) = word;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (t0 + e < o.n) o.tier[t0 + e] = (uint8_t)(word >> (8 * e));
  }
}
// The whole list into the index lists, from the ranks base_r and base_a on.  From the list and not by the thread that found a
// token: one store per 64 entries instead of up to eight masked ones before the list is whole (8192 tokens, 8 heads: selections'
// end to the list 1.35 us instead of 1.7, with the one scan instead of two).
template <int NT>
__device__ __forceinline__ void store_indices(const EmitTarget& o, const int* list, int own_r, int own_a, int base_r, int base_a) {
  for (int i = threadIdx.x; i < own_r + own_a; i += NT) {
    const bool r = i < own_r;
    const int at = r ? base_r + i : base_a + i - own_r;
    if (at < (r ? o.n_retain : o.n_approx)) (r ? o.ir : o.ia)[at] = list[i];
  }
}
// Their rows into the packed cache: retained keys, retained values, approximated keys; each set goes to
// consecutive rows.
template <int NT> __device__ __forceinline__ void copy_rows(const GatherParams& g, int h, int n_approx, const int* list, int own_r, int own_a, int base_r, int base_a) {
  const int pieces = g.row_bytes / 16, log_pieces = 31 - __clz(pieces);
  const int64_t hs = g.hps ? h / g.hps : 0, hh = g.hps ? h % g.hps : h;
  const unsigned char* k_head = g.k + hs * g.k_sb + hh * g.k_sh;
  const unsigned char* v_head = g.v + hs * g.v_sb + hh * g.v_sh;
  unsigned char* k_ret = g.k_ret + ((size_t)h * g.cap_retain + base_r) * g.row_bytes;
  unsigned char* v_ret = g.v_ret + ((size_t)h * g.cap_retain + base_r) * g.row_bytes;
  unsigned char* k_apx = g.k_apx + ((size_t)h * n_approx + base_a) * g.row_bytes;
  const int items = (2 * own_r + own_a) << log_pieces;
  constexpr int U = 4;
  for (int i0 = threadIdx.x; i0 < items; i0 += NT * U) {
    u32x4 x[U];
    unsigned char* to[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = min(i0 + u * NT, items - 1);
      const int row = i >> log_pieces, piece = i & (pieces - 1);
      const bool is_v = row >= own_r && row < 2 * own_r, is_a = row >= 2 * own_r;
      const int t = list[is_v || is_a ? row - own_r : row];
      const unsigned char* from = (is_v ? v_head + (int64_t)t * g.v_st : k_head + (int64_t)t * g.k_st) + piece * 16;
      to[u] = (is_v ? v_ret + (size_t)(row - own_r) * g.row_bytes
                    : (is_a ? k_apx + (size_t)(row - 2 * own_r) * g.row_bytes : k_ret + (size_t)row * g.row_bytes)) + piece * 16;
      x[u] = *reinterpret_cast<const u32x4*>(from);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (i0 + u * NT < items) *reinterpret_cast<u32x4*>(to[u]) = x[u];
  }
}

}  // namespace

}  // namespace vec
