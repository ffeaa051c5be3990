// Three-way routing (Section 3.2, Steps 1 and 3) and compaction into the packed cache, for heads longer than
// route_head.hip takes.  Two launches, synchronised by the kernel boundary only:
//
//   route_bucket_kernel  grid (chunk, head).  Groups a chunk's (score key, token, residual key) entries by the
//                        leading digit of the score key, highest digit first, next to the table
//                        D[b] = #keys of the chunk with digit >= b.  The POOL variant first forms
//                        the score itself, the pooling of the attention mass (Step 1's base scorer).
//   route_list_kernel    grid (part, head).  Every workgroup sums the D tables of its head: the
//                        leading digit of the pool's threshold is the bin where the sum crosses n_pool.
//                        What lies in front of that bin in the chunks' lists is in the pool, what lies in
//                        it (a few hundred entries) is ranked; then the residual keys of the pool, which
//                        the lists carry along, give the second threshold.  All workgroups of a head
//                        find the same two thresholds; each then emits its own part of the tokens (tiers,
//                        ascending index lists) and copies their rows.
//
// A launch costs 4 us before it does anything and the first reads of a workgroup depend on each other, so
// what the workgroups of a head repeat (the pool's residuals, a tenth of the tokens) is cheaper than another launch to
// share it.  32768 tokens x 8 heads take 8 + 21 us (with launches for the pool, for its split and for the rows 40),
// 131072 tokens 13 + 40 (65; rows 16 of the 40), 49157 given scores 7 + 18 (36).
// Bound: latency of dependent reads and barriers; the rows run at 5 TB/s.
//
// Every slot of an output comes from an ordered prefix sum (ties go to the lower token index);
// atomics only feed LDS histograms and the order inside a bucket, which no result depends on.
// No workgroup waits for another inside a kernel.
//
// gather_rows_kernel: row gather k_ret / v_ret / k_apx by the index lists.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "route_common.hpp"

namespace vec {

namespace {

constexpr int kBins = 2048;
constexpr int kTableStride = kBins + 8;   // 16-bit entries of a D table: D[0 .. 2048] and padding to 16 bytes
constexpr int EPT = 4;                    // consecutive elements per thread and tile (one 16-byte load)
constexpr int kStageTokens = 4096;        // a chunk's bucket list is put together in LDS up to this length
constexpr int kMinChunk = 2048;           // tokens per chunk: doubled until a head has at most kMaxChunks
constexpr int kMaxChunks = 32;

// hist[digit] += cnt (cnt in 0..7) for every lane.  Keys of neighbouring tokens often share their
// leading bits, so a plain LDS atomic would serialise up to 64 lanes on one bin: lanes that agree
// with a leader are merged through ballots of the three bits of cnt and added by the leader alone;
// after two rounds the stragglers (few, spread over bins) add themselves.
__device__ __forceinline__ void hist_add_weighted(int* hist, uint32_t digit, int cnt, int lane) {
  unsigned long long todo = __ballot(cnt > 0);
#pragma unroll
  for (int round = 0; round < 2; ++round) {
    if (todo == 0) return;
    const int leader = __ffsll((long long)todo) - 1;
    const uint32_t d = __builtin_amdgcn_readlane(digit, leader);
    const bool match = cnt > 0 && digit == d;
    const unsigned long long b0 = __ballot(match && (cnt & 1)), b1 = __ballot(match && (cnt & 2)),
                             b2 = __ballot(match && (cnt & 4));
    if (lane == leader) atomicAdd(&hist[d], __popcll(b0) + 2 * __popcll(b1) + 4 * __popcll(b2));
    if (match) cnt = 0;
    todo &= ~(b0 | b1 | b2);
  }
  if (cnt > 0) atomicAdd(&hist[digit], cnt);
}

// Leading digits of a thread's EPT consecutive keys into an LDS histogram: the keys that agree
// with the thread's first valid one go in together, the others one by one.
__device__ __forceinline__ void hist_add_thread_keys(int* hist, const uint32_t (&key)[EPT], const bool (&ok)[EPT], int lane,
                                                     const DigitMap& map) {
  uint32_t dg[EPT];
#pragma unroll
  for (int j = 0; j < EPT; ++j) dg[j] = map.digit(key[j]);
  // lanes that mostly go elsewhere than the first one: every key for itself
  if (__popcll(__ballot(ok[0] && dg[0] == (uint32_t)__builtin_amdgcn_readfirstlane((int)dg[0]))) <= 8) {      // uniform
#pragma unroll
    for (int j = 0; j < EPT; ++j)
      if (ok[j]) atomicAdd(&hist[dg[j]], 1);
    return;
  }
  int first = -1;
#pragma unroll
  for (int j = EPT - 1; j >= 0; --j)
    if (ok[j]) first = j;
  const uint32_t d0 = first >= 0 ? dg[first] : 0u;
  int cnt = 0;
#pragma unroll
  for (int j = 0; j < EPT; ++j) cnt += ok[j] && dg[j] == d0;
  hist_add_weighted(hist, d0, cnt, lane);
#pragma unroll
  for (int j = 0; j < EPT; ++j)
    if (ok[j] && dg[j] != d0) atomicAdd(&hist[dg[j]], 1);
}

// ---------------------------------------------------------------------------
// prefix sums: inside a wave on the DPP network, across the waves through one LDS row that
// every thread reads whole (no chain of dependent LDS reads)
// ---------------------------------------------------------------------------
// NW per-wave values -> their sum over the waves before `wave`, and over all waves
template <int NW> __device__ __forceinline__ void wave_row_sums(const int* row, int wave, int& before, int& total) {
  before = 0;
  total = 0;
#pragma unroll
  for (int q = 0; q < NW; ++q) {
    const int x = row[q];
    total += x;
    before += (q < wave) ? x : 0;
  }
}

// Counts of a 2048-bin LDS histogram -> D[b] = #(digit >= b), written as a 16-bit table to
// global memory (D[2048] = 0 and the padding included); the histogram itself is turned into
// #(digit > b), the first slot of bin b when the keys are laid out highest digit first.
// NT threads, thread t owns the kBins / NT bins below and including kBins - 1 - t * kBins / NT.
// row: LDS, NT / 64 ints.  Ends with a barrier.
template <int NT>
__device__ __forceinline__ void counts_to_table(int* hist, uint16_t* table, int* row) {
  constexpr int BPT = kBins / NT, NW = NT / kWave;
  static_assert(BPT % 2 == 0, "pairs of bins are stored as one word");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int hi = kBins - 1 - BPT * (int)threadIdx.x;
  int c[BPT], s[BPT], run = 0;
#pragma unroll
  for (int k = 0; k < BPT; ++k) { c[k] = hist[hi - k]; run += c[k]; s[k] = run; }
  const int incl = wave_incl_scan_dpp(run);
  if (lane == 63) row[wave] = incl;
  __syncthreads();
  int before, total;
  wave_row_sums<NW>(row, wave, before, total);
  before += incl - run;
  uint32_t* t32 = reinterpret_cast<uint32_t*>(table);
#pragma unroll
  for (int k = 0; k < BPT; k += 2) {          // bins hi-k (odd) and hi-k-1 (even) share a word
    const uint32_t d_hi = (uint32_t)(before + s[k]), d_lo = (uint32_t)(before + s[k + 1]);
    t32[(hi - k - 1) >> 1] = d_lo | (d_hi << 16);
    hist[hi - k] = before + s[k] - c[k];
    hist[hi - k - 1] = before + s[k + 1] - c[k + 1];
  }
  if (threadIdx.x < (kTableStride - kBins) / 2) t32[kBins / 2 + threadIdx.x] = 0u;
  __syncthreads();
}

// ---------------------------------------------------------------------------
// buckets of the score keys by leading digit (and, POOL, the pooled score itself)
// ---------------------------------------------------------------------------
struct BucketParams {
  const float* src;       // POOL: attention mass [H, n]; otherwise the scores [H, n]
  float* score;           // POOL: output [H, n]
  uint16_t* table;        // [H, C, kTableStride] or null (POOL only: pooling alone)
  uint32_t* bkey;         // [H, n]: chunk c owns [c * chunk_tokens, ...), keys grouped by digit, highest first
  int32_t* bpos;          // [H, n]: the token each key belongs to
  uint32_t* beps;         // [H, n]: and its residual key (smaller residual, larger key)
  const float* eps;       // [H, n] residuals
  int n, n_prefix, kernel, chunk_tokens, n_chunks;
  float inv_kernel;       // POOL: 1 / kernel
  int take_max;           // POOL: the window's largest mass instead of its sum over the kernel size
  const float4* range;    // [H, n_range] (count, sum l, sum l * l) of the mass left by the scorer's workgroups, when n_range > 0
  int n_range;
  float log_ref;          // what the scorer subtracted from log2(mass)
  const BucketParams* seq_table;   // RAGGED launches: the sequences' parameter blocks, seq_hps heads each
  int seq_hps;
};

// Chunks of 2048 tokens: 512 threads; longer ones 1024, so that those of up to 4096 are one tile too.  What bounds it is
// latency: statistics, inputs, a histogram, a scan, the scatter.  The inputs travel while the statistics are turned into the
// map, by 16-byte loads at any element (a head whose length is no multiple of four took an element at a time: 20011
// tokens x 8 heads 2 us more).
template <int BT, bool POOL, bool RAGGED = false>
__global__ __launch_bounds__(BT) void route_bucket_kernel(KernelArgs<BucketParams, RAGGED> args) {
  BucketParams p = args.p;
  int chunk, h;
  xcd_chunk_head(chunk, h);
  take_sequence<RAGGED>(p, h);
  if (chunk >= p.n_chunks) return;
  __shared__ int hist[kBins];
  __shared__ int row[BT / kWave];
  __shared__ uint32_t sample[BT / kWave][4];
  __shared__ __align__(16) uint32_t stage_key[kStageTokens];
  __shared__ __align__(16) int32_t stage_pos[kStageTokens];
  __shared__ __align__(16) uint32_t stage_eps[kStageTokens];
  const int lane = threadIdx.x & 63;
  const bool do_buckets = p.table != nullptr;
  DigitMap map = {0u, 21};
  // every wave adds up the head's statistics itself (in one fixed order), so all workgroups of
  // the head cut the same buckets
  constexpr int kRangeRegs = 2;
  float4 range_x[kRangeRegs];
  if (do_buckets && p.n_range > 0) {
    const float4* r = p.range + (size_t)h * p.n_range;
#pragma unroll
    for (int u = 0; u < kRangeRegs; ++u) {
      const int i = u * kWave + lane;
      range_x[u] = i < p.n_range ? r[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  const float* src = p.src + (size_t)h * p.n;
  const int begin = chunk * p.chunk_tokens, end = min(p.n, begin + p.chunk_tokens);
  constexpr int kBucketTile = BT * EPT;
  // tokens t .. t + 3 of a head's array; 0 outside [first, stop)
  auto load4 = [&](const float* a, int t, int first, int stop) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (t >= first && t + 4 <= stop) {
      x = *reinterpret_cast<const f32x4_u*>(a + t);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t + e >= first && t + e < stop) x[e] = a[t + e];
    }
    return x;
  };
  const float* scores = POOL ? p.score + (size_t)h * p.n : src;
  const float* eps = do_buckets ? p.eps + (size_t)h * p.n : nullptr;
  // The first tile's inputs are requested before the statistics are turned into the map: the masses around the thread's
  // four tokens (POOL: enough for kernels of up to 9, the usual ones), or the scores; and the residuals.
  const int half = POOL ? p.kernel / 2 : 0;
  constexpr int kNear = POOL ? 3 : 1;
  const int first_t0 = begin + (int)threadIdx.x * EPT;
  f32x4 near0[kNear], eps0 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < kNear; ++q) near0[q] = load4(src, first_t0 + (q - kNear / 2) * EPT, 0, POOL ? p.n : end);
  if (do_buckets) eps0 = load4(eps, first_t0, 0, end);
  if (do_buckets) {
    for (int i = threadIdx.x; i < kBins; i += BT) hist[i] = 0;
    if (p.n_range > 0) {
      float cnt = 0.f, sl = 0.f, sll = 0.f;
#pragma unroll
      for (int u = 0; u < kRangeRegs; ++u) { cnt += range_x[u].x; sl += range_x[u].y; sll += range_x[u].z; }
      const float4* r = p.range + (size_t)h * p.n_range;
      for (int i = kRangeRegs * kWave + lane; i < p.n_range; i += kWave) {       // long sequences only
        const float4 x = r[i];
        cnt += x.x; sl += x.y; sll += x.z;
      }
      map = digit_map_for_stats(wave_sum_dpp(cnt), wave_sum_dpp(sl), wave_sum_dpp(sll), p.log_ref);
    }
    if (!POOL) {
      // no statistics came with the scores: four keys out of every 256, the same sample in every
      // workgroup of the head (integer sums: any order gives the same map)
      uint32_t c = 0, s1 = 0, s2lo = 0, s2hi = 0;
      const bool al = (((size_t)h * p.n) & 3) == 0 && (reinterpret_cast<uintptr_t>(p.src) & 15u) == 0;
      for (int i = (int)threadIdx.x * 256; i < p.n; i += BT * 256) {
        float x[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
        if (al && i + 4 <= p.n) {
          const float4 v = *reinterpret_cast<const float4*>(src + i);
          x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (i + j < p.n) x[j] = src[i + j];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t key = float_key(x[j]);
          if (key > 0x007fffffu && key < 0xff800000u) {                     // finite
            const unsigned long long k = key >> 12, kk = k * k;
            c += 1; s1 += (uint32_t)k; s2lo += (uint32_t)(kk & 0xfffffu); s2hi += (uint32_t)(kk >> 20);
          }
        }
      }
      const int wave = threadIdx.x >> 6;
      c = (uint32_t)wave_total_of_scan(wave_incl_scan_dpp((int)c));
      s1 = (uint32_t)wave_total_of_scan(wave_incl_scan_dpp((int)s1));
      s2lo = (uint32_t)wave_total_of_scan(wave_incl_scan_dpp((int)s2lo));
      s2hi = (uint32_t)wave_total_of_scan(wave_incl_scan_dpp((int)s2hi));
      if (lane == 0) { sample[wave][0] = c; sample[wave][1] = s1; sample[wave][2] = s2lo; sample[wave][3] = s2hi; }
      __syncthreads();
      unsigned long long tc = 0, t1 = 0, t2 = 0;
#pragma unroll
      for (int w = 0; w < BT / kWave; ++w) {
        tc += sample[w][0]; t1 += sample[w][1];
        t2 += (unsigned long long)sample[w][2] + ((unsigned long long)sample[w][3] << 20);
      }
      map = digit_map_for_sample(tc, t1, t2);
    }
    __syncthreads();
  }
  uint32_t key0[EPT];                            // the keys of the first tile stay in registers for the scatter
  for (int tile = begin; tile < end; tile += kBucketTile) {        // uniform trip count: whole waves take part
    const int t0 = tile + (int)threadIdx.x * EPT;
    float s[EPT];
    bool ok[EPT];
#pragma unroll
    for (int j = 0; j < EPT; ++j) ok[j] = t0 + j < end;
    if (POOL) {
      // windows of 2 half + 1 masses, folded in ascending token order over the prefix columns; mass is never
      // negative, so the sums and maxima may start from zero
      auto fold = [&](auto quads_tag, const f32x4* m) {
        constexpr int Q = decltype(quads_tag)::value;        // quads on either side
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
          float acc = 0.f;
#pragma unroll
          for (int d = -Q * EPT; d <= Q * EPT; ++d) {
            const int at = Q * EPT + j + d;
            if (d >= -half && d <= half && t0 + j + d < p.n_prefix) acc = p.take_max ? fmaxf(acc, m[at >> 2][at & 3]) : acc + m[at >> 2][at & 3];
          }
          s[j] = acc;
        }
      };
      if (half <= EPT) {
        f32x4 m[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) m[q] = tile == begin ? near0[q] : load4(src, t0 + (q - 1) * EPT, 0, p.n);
        fold(std::integral_constant<int, 1>{}, m);
      } else if (half <= 2 * EPT) {
        f32x4 m[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) m[q] = load4(src, t0 + (q - 2) * EPT, 0, p.n);
        fold(std::integral_constant<int, 2>{}, m);
      } else {
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
          const int t = t0 + j, lo = max(0, t - half), hi = min(p.n_prefix - 1, t + half);
          float acc = 0.f;
          if (ok[j])
            for (int i = lo; i <= hi; ++i) acc = p.take_max ? fmaxf(acc, src[i]) : acc + src[i];
          s[j] = acc;
        }
      }
      float* dst = p.score + (size_t)h * p.n;
#pragma unroll
      for (int j = 0; j < EPT; ++j) {
        if (!p.take_max) s[j] = pool_mean(s[j], (float)p.kernel, p.inv_kernel);
        if (!ok[j] || t0 + j >= p.n_prefix) s[j] = INFINITY;         // window columns
      }
      if (ok[EPT - 1]) {
        const f32x4 x = {s[0], s[1], s[2], s[3]};
        *reinterpret_cast<f32x4_u*>(dst + t0) = x;
      } else {
#pragma unroll
        for (int j = 0; j < EPT; ++j)
          if (ok[j]) dst[t0 + j] = s[j];
      }
    } else {
      const f32x4 x = tile == begin ? near0[0] : load4(scores, t0, 0, end);
#pragma unroll
      for (int j = 0; j < EPT; ++j) s[j] = x[j];
    }
    if (do_buckets) {
      uint32_t key[EPT];
#pragma unroll
      for (int j = 0; j < EPT; ++j) key[j] = float_key(s[j]);
      hist_add_thread_keys(hist, key, ok, lane, map);
      if (tile == begin) {
#pragma unroll
        for (int j = 0; j < EPT; ++j) key0[j] = key[j];
      }
    }
  }
  if (!do_buckets) return;
  __syncthreads();
  counts_to_table<BT>(hist, p.table + ((size_t)h * p.n_chunks + chunk) * kTableStride, row);
  // scatter: hist[b] is now the next free slot of bin b in the chunk's list
  // The slots of neighbouring tokens are far apart in the list (the finer the buckets, the farther),
  // so the list of a chunk that fits is put together in LDS and written out in order; longer
  // chunks scatter their entries straight to memory.
  uint32_t* bkey = p.bkey + (size_t)h * p.n + begin;
  int32_t* bpos = p.bpos + (size_t)h * p.n + begin;
  uint32_t* beps = p.beps + (size_t)h * p.n + begin;
  const bool staged = p.chunk_tokens <= kStageTokens;
  for (int tile = begin; tile < end; tile += kBucketTile) {
    const int t0 = tile + (int)threadIdx.x * EPT;
    uint32_t key[EPT];
    f32x4 ev = eps0;
    if (tile == begin) {
#pragma unroll
      for (int j = 0; j < EPT; ++j) key[j] = key0[j];
    } else {                                     // later tiles: the scores this thread stored (or read) above
      const f32x4 x = load4(scores, t0, 0, end);
      ev = load4(eps, t0, 0, end);
#pragma unroll
      for (int j = 0; j < EPT; ++j) key[j] = float_key(x[j]);
    }
#pragma unroll
    for (int j = 0; j < EPT; ++j) {
      if (t0 + j < end) {
        const int slot = atomicAdd(&hist[map.digit(key[j])], 1);
        if (slot < end - begin) {                                                // always true: counted above
          const uint32_t ek = ~float_key(ev[j]);
          if (staged) { stage_key[slot] = key[j]; stage_pos[slot] = t0 + j; stage_eps[slot] = ek; }
          else { bkey[slot] = key[j]; bpos[slot] = t0 + j; beps[slot] = ek; }
        }
      }
    }
  }
  if (staged) {                                  // the list leaves LDS in order: whole cache lines per wave
    __syncthreads();
    const int cnt = end - begin;
    if ((((size_t)h * p.n) & 3) == 0) {
      for (int i = (int)threadIdx.x * 4; i < cnt; i += BT * 4) {
        if (i + 4 <= cnt) {
          *reinterpret_cast<uint4*>(bkey + i) = *reinterpret_cast<const uint4*>(stage_key + i);
          *reinterpret_cast<int4*>(bpos + i) = *reinterpret_cast<const int4*>(stage_pos + i);
          *reinterpret_cast<uint4*>(beps + i) = *reinterpret_cast<const uint4*>(stage_eps + i);
        } else {
          for (int j = i; j < cnt; ++j) { bkey[j] = stage_key[j]; bpos[j] = stage_pos[j]; beps[j] = stage_eps[j]; }
        }
      }
    } else {
      for (int i = threadIdx.x; i < cnt; i += BT) { bkey[i] = stage_key[i]; bpos[i] = stage_pos[i]; beps[i] = stage_eps[i]; }
    }
  }
}

// ---------------------------------------------------------------------------
// both selections, emission, rows
// ---------------------------------------------------------------------------
struct RouteParams {
  const float* score; const float* eps;
  int n, n_pool, n_approx;
  int chunk_tokens, n_chunks;      // of the bucket lists
  int part_tokens;                 // tokens per workgroup
  const uint16_t* table;           // [H, C, kTableStride] leading digits of the score keys
  const uint32_t* bkey;            // [H, n] score keys grouped by leading digit, chunk by chunk
  const int32_t* bpos;             // their tokens
  const uint32_t* beps;            // and residual keys
  uint8_t* tier; int32_t* idx_retain; int32_t* idx_approx;
  GatherParams g;                  // row copies (k null: none)
  const RouteParams* seq_table;    // RAGGED launches: the sequences' parameter blocks, seq_hps heads each
  int seq_hps;
};

// Threads of the list kernel: every workgroup works through the head's pool, so sixteen waves share it (the routing of
// 8 heads, sixteen waves against eight, in us: 20.0 / 20.4 at 32768 tokens, 24.5 / 25.9 at 65536, 34.5 / 38.3 at 131072).
constexpr int HT = 1024;
constexpr int HW = kWaves<HT>;
constexpr int kHeadBlock = kBlock<HT>;
constexpr int kTableGroups = kBins / 8;  // of eight bins
constexpr int kMaxGroups = HT;           // as many as the registers of a workgroup hold, at most

// Per chunk a run of the head's lists: its first entry, its length, and the groups of kRunGroup entries before it
struct Runs {
  int at[kMaxChunks], count[kMaxChunks], group_start[kMaxChunks], n_groups;
};
constexpr int kRunGroup = 4 * kWave;     // entries that a wave takes at a time

struct ListShared {
  __align__(16) int hist[kHeadBins];
  __align__(16) int list[kHeadBlock];    // tokens whose rows this workgroup copies: retained, then approximated
  int coarse[HT / kTableGroups][kTableGroups + 2];      // sums of the tables at every eighth bin, the highest first, over every fourth chunk
  __align__(16) uint16_t digit[kMaxChunks][16];         // the chosen eight bins' entries of every chunk's table, and the next bin's
  // per chunk: entries in front of the chosen bin, the groups of 64 of them before the chunk's, the entries
  // of the bin (candidates) before the chunk's, and the chunk's own
  int front[kMaxChunks], group_start[kMaxChunks], cand_start[kMaxChunks], cand_count[kMaxChunks];
  int n_groups;
  // runs of entries that do not fit the registers: candidates; entries in front of the bin, [1] all or [0] the rest
  Runs cand_runs, front_runs[2];
  int2 run_group[HT];                    // for walk_runs
  int2 group[kMaxGroups];                // the first groups: place of the first entry in the head's lists, number of entries
  __align__(16) uint32_t cand[kRankCap];
  int wsum[3][HW];
  float stat[3][HW];
  uint32_t range[2][HW];
  uint32_t center[2];
  int pick[3];
  int n_cand;
  uint32_t thr;
  int quota, equal;
};

// Lane c of one wave holds chunk c's numbers of entries in front of the bin and in it (0 beyond the chunks)
__device__ __forceinline__ void leave_chunk_counts(int front, int cnt, int n_chunks, ListShared& sh) {
  const int lane = threadIdx.x & 63, groups = (front + 63) >> 6;
  const int g_incl = wave_incl_scan_dpp(groups), c_incl = wave_incl_scan_dpp(cnt);
  if (lane < kMaxChunks) {
    sh.front[lane] = front;
    sh.group_start[lane] = lane < n_chunks ? g_incl - groups : 0x7fffffff;
    sh.cand_start[lane] = lane < n_chunks ? c_incl - cnt : 0x7fffffff;
    sh.cand_count[lane] = cnt;
  }
  if (lane == 63) sh.n_groups = g_incl;
}
// the same for a run of every chunk (count 0 beyond the chunks)
__device__ __forceinline__ void leave_runs(int at, int count, int n_chunks, Runs& r) {
  const int lane = threadIdx.x & 63, groups = (count + kRunGroup - 1) / kRunGroup;
  const int incl = wave_incl_scan_dpp(groups);
  if (lane < kMaxChunks) { r.at[lane] = at; r.count[lane] = count; r.group_start[lane] = lane < n_chunks ? incl - groups : 0x7fffffff; }
  if (lane == 63) r.n_groups = incl;
}

// Leading digit of the k-th largest key of a head from the D tables of its chunks: summed over the
// chunks, S[b] = #(digit >= b) falls from the key count at b = 0 to 0 at b = 2048, and the digit is
// the one bin with S[b+1] < k <= S[b].  What this costs is load instructions (16 cycles of a CU's address unit each,
// however narrow) and trips to memory.  So a thread takes eight bins of every fourth chunk, 16 bytes a load and all in
// one trip; the threads whose bins hold k, and those that hold the next bin up, leave their chunks' entries in LDS,
// where lane c of wave 0 finds chunk c's: that gives the digit, and where every chunk keeps its entries.  (With two bytes
// of every table per load and a second trip for the digit, routing and rows of 49157 given scores took 37.6 us, now 35.5.)
// prefetch() is called once the loads are out.
// k lies between 1 and the number of keys (launch_route refuses any other n_pool, and every key is in one bin), so exactly one
// bin holds it: sh.digit is read where it was written.
template <typename Prefetch>
__device__ __forceinline__ void pick_from_tables(const uint16_t* tables, int n_chunks, int k, ListShared& sh, Prefetch prefetch) {
  constexpr int kPer = HT / kTableGroups, kLoads = kMaxChunks / kPer;      // chunks taken side by side, one after the other
  static_assert(HT % kTableGroups == 0 && kMaxChunks % kPer == 0 && kTableGroups % kWave == 0, "whole waves on a chunk");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = (int)threadIdx.x % kTableGroups, first = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kTableGroups);
  const int lo = kBins - 8 - 8 * t;             // the thread's bins: lo .. lo + 7
  u32x4 e[2][kLoads / 2];
  auto load_half = [&](int v) {
#pragma unroll
    for (int u = 0; u < kLoads / 2; ++u)
      e[v][u] = *reinterpret_cast<const u32x4*>(tables + (size_t)min(first + (v * (kLoads / 2) + u) * kPer, n_chunks - 1) * kTableStride + lo);
  };
  load_half(0);
#pragma unroll
  for (int u = 0; u < kLoads / 2; ++u) e[1][u] = u32x4{0u, 0u, 0u, 0u};
  if (n_chunks > kMaxChunks / 2) load_half(1);  // uniform
  prefetch();
  int own = 0;                                  // S[lo] over the thread's chunks
#pragma unroll
  for (int u = 0; u < kLoads; ++u)
    if (first + u * kPer < n_chunks) own += (int)(e[u / (kLoads / 2)][u % (kLoads / 2)][0] & 0xffffu);
  sh.coarse[first][t + 1] = own;
  if ((int)threadIdx.x < kPer) { sh.coarse[threadIdx.x][0] = 0; sh.coarse[threadIdx.x][kTableGroups + 1] = 0; }
  if (threadIdx.x == 0) sh.pick[0] = 0;
  lds_barrier();
  int above = 0, here = 0, below = 0;           // S[lo + 8], S[lo], S[lo - 8]
#pragma unroll
  for (int q = 0; q < kPer; ++q) { above += sh.coarse[q][t]; here += sh.coarse[q][t + 1]; below += sh.coarse[q][t + 2]; }
  if (above < k && k <= here) {
    sh.pick[0] = lo;
#pragma unroll
    for (int u = 0; u < kLoads; ++u)
      *reinterpret_cast<u32x4*>(&sh.digit[first + u * kPer][0]) = e[u / (kLoads / 2)][u % (kLoads / 2)];
  } else if (here < k && k <= below) {          // k is in the eight bins below: their upper end is this thread's
#pragma unroll
    for (int u = 0; u < kLoads; ++u) sh.digit[first + u * kPer][8] = (uint16_t)(e[u / (kLoads / 2)][u % (kLoads / 2)][0] & 0xffffu);
  }
  lds_barrier();
  if (wave == 0) {
    const int at = sh.pick[0];
    int d[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) d[q] = 0;
    if (lane < n_chunks) {
      const u32x4 x = *reinterpret_cast<const u32x4*>(&sh.digit[lane][0]);
#pragma unroll
      for (int q = 0; q < 8; ++q) d[q] = (int)((x[q / 2] >> (16 * (q % 2))) & 0xffffu);
      d[8] = at + 8 < kBins ? sh.digit[lane][8] : 0;
    }
    int S[9], j = 0;
#pragma unroll
    for (int q = 0; q < 9; ++q) S[q] = wave_total_of_scan(wave_incl_scan_dpp(d[q]));
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (S[q + 1] < k && k <= S[q]) j = q;
    int front = d[1], cnt = d[0] - d[1], in_front = S[1], count = S[0] - S[1];
#pragma unroll
    for (int q = 1; q < 8; ++q)
      if (j == q) { front = d[q + 1]; cnt = d[q] - d[q + 1]; in_front = S[q + 1]; count = S[q] - S[q + 1]; }
    leave_chunk_counts(front, cnt, n_chunks, sh);
    if (lane == 0) { sh.pick[0] = at + j; sh.pick[1] = in_front; sh.pick[2] = count; }
  }
  lds_barrier();
}

// the chunk whose entries hold number idx of a concatenation (start: [kMaxChunks], ascending)
__device__ __forceinline__ int chunk_of(const int* start, int idx) {
  int c = 0;
#pragma unroll
  for (int s = kMaxChunks / 2; s > 0; s >>= 1)
    if (start[c + s] <= idx) c += s;
  return c;
}

// The runs of chunks [c0, c1): use(load(place in the head's lists), e) for e = 0 .. 3, the entries at that place and
// behind it.  A wave takes kRunGroup entries of a run at a time, four neighbours per lane, and has U such groups on
// their way; the groups' places are laid out by the threads, one each.  At a run's end the lanes read from four before
// the end on and skip what another lane has, so a run of fewer than four reads up to three entries in front of it
// (at the very first place: the end of the array before, see route_layout).  Whole workgroup.  An entry per lane
// and a look-up of the chunk per group took three times as long (131072 tokens x 8 heads, 64 scores a few ulps
// apart: 360 us for the routing, now 214).
template <int U, typename Load, typename Use>
__device__ __forceinline__ void walk_runs(const Runs& runs, int2* table, int n_chunks, int c0, int c1, Load load, Use use) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int g0 = __builtin_amdgcn_readfirstlane(runs.group_start[c0]);
  const int g1 = __builtin_amdgcn_readfirstlane(c1 < n_chunks ? runs.group_start[c1] : runs.n_groups);
  for (int r = g0; r < g1; r += HT) {
    const int g = r + (int)threadIdx.x, count = min(HT, g1 - r);
    lds_barrier();
    if (g < g1) {
      const int c = chunk_of(runs.group_start, g), first = (g - runs.group_start[c]) * kRunGroup;
      table[threadIdx.x] = make_int2(runs.at[c] + first, min(kRunGroup, runs.count[c] - first));
    }
    lds_barrier();
    for (int i = wave; i < count; i += U * HW) {
      decltype(load(0)) x[U];
      int skip[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int2 at = table[min(i + u * HW, count - 1)];
        const int first = min(4 * lane, at.y - 4);
        x[u] = load(at.x + first);
        skip[u] = i + u * HW < count ? 4 * lane - first : 4;
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e >= skip[u]) use(x[u], e);
    }
  }
}
__device__ __forceinline__ u32x4 load_entries(const void* list, int at) {
  return *reinterpret_cast<const u32x4_u*>(reinterpret_cast<const uint32_t*>(list) + at);
}

// The k-th largest key: keys above thr are selected, and of those equal to it the quota with the lowest tokens
// (all_equal: every one).
struct Cut { uint32_t thr; int quota; bool all_equal; };

// A sample of the keys in registers (0: no key), every fourth slot: count, sum and sum of squares in units of 4096
// keys about the center; every wave leaves its own in sh.stat for list_select.
template <int NS>
__device__ __forceinline__ void leave_sample(const uint32_t (&key)[NS], uint32_t center, ListShared& sh) {
  float cnt = 0.f, s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int j = 0; j < NS; j += 4) {
    const bool ok = key[j] > 0x007fffffu && key[j] < 0xff800000u;       // a finite number
    const float dlt = ok ? (float)((int)(key[j] >> 12) - (int)(center >> 12)) : 0.f;
    cnt += ok ? 1.f : 0.f;
    s1 += dlt;
    s2 = fmaf(dlt, dlt, s2);
  }
  cnt = wave_sum_dpp(cnt); s1 = wave_sum_dpp(s1); s2 = wave_sum_dpp(s2);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { sh.stat[0][wave] = cnt; sh.stat[1][wave] = s1; sh.stat[2][wave] = s2; }
}

// Among the keys in registers (0: no key) and those that more(f) hands to f; 1 <= k <= number of keys.
// total: number of keys, all in [lo, lo + span]; center: what leave_sample was given, or tight: the range starts and
// ends with a key (then no sample is needed).  MORE_IS_TIGHT: more() has none where the range is not tight.  The
// caller has passed a barrier since the last use of sh but for the sample.
template <bool MORE_IS_TIGHT, int NS, typename More>
__device__ __forceinline__ Cut list_select(const uint32_t (&key)[NS], More more, int total, int k, uint32_t center, bool tight, uint32_t lo,
                                           uint32_t span, ListShared& sh) {
  const int lane = threadIdx.x & 63;
  auto each = [&](auto f) {
#pragma unroll
    for (int i = 0; i < NS; ++i) f(key[i]);
    more(f);
  };
  auto each_first = [&](auto f) {
#pragma unroll
    for (int i = 0; i < NS; ++i) f(key[i]);
    if (!MORE_IS_TIGHT) more(f);
  };
  int count = total;
  if (threadIdx.x == 0) sh.n_cand = 0;
  if ((int)threadIdx.x < kRankCap) sh.cand[threadIdx.x] = 0u;
  if (total > kRankCap && !tight) {                                     // uniform
    clear_bins<HT>(sh.hist);
    lds_barrier();
    const float cnt = sum_of_waves<HT>(sh.stat[0], lane), s1 = sum_of_waves<HT>(sh.stat[1], lane), s2 = sum_of_waves<HT>(sh.stat[2], lane);
    if (!(cnt >= 32.f && s2 == 0.f && around_center<HT>(each_first, center, lo, span, k, count, sh.wsum[0]))) {
      const DigitMap map = digit_map_about(center, cnt, s1, s2);
      each_first([&](uint32_t x) { if (x != 0u) atomicAdd(&sh.hist[map.digit(x)], 1); });
      lds_barrier();
      int d, above;
      pick_bin<HT>(sh.hist, sh.wsum[0], sh.pick, k, d, above, count);
      k -= above;
      bucket_range(map, d, lo, span);
    }
  } else {
    lds_barrier();
  }
  narrow<HT>(each, tight, lo, span, k, count, sh.hist, sh.wsum[0], sh.pick, sh.range);
  if (span == 0u) { lds_barrier(); return {lo, k, count == k}; }        // one key, however many tokens
  auto collect = [&](uint32_t x) {
    if (x - lo <= span) {
      const int at = atomicAdd(&sh.n_cand, 1);
      if (at < kRankCap) sh.cand[at] = x;
    }
  };
  bool any = false;                                                     // few waves have one: a branch per slot only there
#pragma unroll
  for (int i = 0; i < NS; ++i) any |= key[i] - lo <= span;
  if (__any(any)) {
#pragma unroll
    for (int i = 0; i < NS; ++i) collect(key[i]);
  }
  more(collect);
  lds_barrier();
  if ((int)threadIdx.x < count) {
    const uint32_t mine = sh.cand[threadIdx.x];
    int greater = 0, equal = 0;
    for (int j = 0; j < count; j += 16) {                               // the rest of the list is 0: below every key
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint4 x = *reinterpret_cast<const uint4*>(sh.cand + j + 4 * q);
        greater += (x.x > mine) + (x.y > mine) + (x.z > mine) + (x.w > mine);
        equal += (x.x == mine) + (x.y == mine) + (x.z == mine) + (x.w == mine);
      }
    }
    if (greater < k && k <= greater + equal) { sh.thr = mine; sh.quota = k - greater; sh.equal = equal; }     // the same values from every thread that finds it
  }
  lds_barrier();
  return {sh.thr, sh.quota, sh.quota == sh.equal};
}

// The last of the `quota` lowest tokens in [first, last] whose key is thr; each(a, b, f) hands every (key, token) with
// a token in [a, b], and maybe others, to f.
template <typename Each>
__device__ __forceinline__ int token_cut(Each each, uint32_t thr, int quota, int first, int last, ListShared& sh) {
  uint32_t lo = 0u, span = (uint32_t)(last - first);                    // of last - token
  while (span != 0u) {
    const int s = max(0, 21 - (int)__clz(span));
    int d, above, count;
    clear_bins<HT>(sh.hist);
    lds_barrier();
    each(last - (int)(lo + span), last - (int)lo, [&](uint32_t key, int tok) {
      const uint32_t v = (uint32_t)(last - tok) - lo;
      if (key == thr && v <= span) atomicAdd(&sh.hist[v >> s], 1);
    });
    lds_barrier();
    pick_bin<HT>(sh.hist, sh.wsum[0], sh.pick, quota, d, above, count);
    quota -= above;
    lo += (uint32_t)d << s;
    span = min(span - ((uint32_t)d << s), (1u << s) - 1u);
  }
  lds_barrier();
  return last - (int)lo;
}

constexpr int kCandSlots = 2;            // candidates per thread kept in registers

// Where a head's tokens are cut: in_pool() and, inside the pool, is_approx(), of order-preserving keys and tokens; and how
// many of the pool, and of its approximated tokens, this thread found in the chunks before the workgroup's own
// (counts of whole waves in lane 0).
struct HeadCut {
  uint32_t top_thr, low_thr;
  int top_tok, low_tok;                  // the last token that an equal key is taken of
  bool any_approx;
  int pool_before, apx_before;
  __device__ __forceinline__ bool in_pool(uint32_t key, int tok) const { return key > top_thr || (key == top_thr && tok <= top_tok); }
  __device__ __forceinline__ bool is_approx(uint32_t key, int tok) const {
    return any_approx && (key > low_thr || (key == low_thr && tok <= low_tok));
  }
};

// Both selections of a head, by every workgroup of it.  SLOTS: pool members per thread kept in registers.  ALL: they and
// the candidates all fit; otherwise the rest is read again for every pass over it.  The two are apart because the
// passes over what does not fit would lie between the others in the instruction cache (one code for both: 0.3 to 3 us
// more for heads that fit).
template <int SLOTS, bool ALL>
__device__ __forceinline__ HeadCut cut_head(const RouteParams& p, int h, int own_chunk, ListShared& sh) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), tid = threadIdx.x, n = p.n;
  const uint32_t* bkey = p.bkey + (size_t)h * n;
  const int32_t* bpos = p.bpos + (size_t)h * n;
  const uint32_t* beps = p.beps + (size_t)h * n;
  auto keys_at = [&](int at) { return load_entries(bkey, at); };
  struct Tokens { u32x4 key, tok; };
  struct Entries { u32x4 key, tok, eps; };
  int n_front = __builtin_amdgcn_readfirstlane(sh.pick[1]), n_cand = __builtin_amdgcn_readfirstlane(sh.pick[2]);
  // More candidates than the registers hold: their range first.  If all are one number (a plateau of scores), those
  // of the lowest tokens are in the pool: whole chunks, which join the entries in front of the bin, and a part of
  // one chunk, whose candidates stay.
  uint32_t least = 1u, most = 0xffffffffu;
  bool plateau = false;
  int cut_chunk = 0;
  const bool all_candidates = p.n_pool - n_front == n_cand;            // are in the pool
  if (!ALL && n_cand > kCandSlots * HT) {                              // uniform
    int front = 0, cnt = 0;
    if (lane < p.n_chunks) { front = sh.front[lane]; cnt = sh.cand_count[lane]; }
    if (wave == 0) leave_runs(lane * p.chunk_tokens + front, cnt, p.n_chunks, sh.cand_runs);
    lds_barrier();
    key_range<HT>([&](auto f) { walk_runs<4>(sh.cand_runs, sh.run_group, p.n_chunks, 0, p.n_chunks, keys_at, [&](u32x4 x, int e) { f(x[e]); }); }, least,
              most - least, sh.range, least, most);
    plateau = least == most;
    if (plateau) {
      cut_chunk = __builtin_amdgcn_readfirstlane(chunk_of(sh.cand_start, p.n_pool - n_front - 1));
      n_front += __builtin_amdgcn_readfirstlane(sh.cand_start[cut_chunk]);
      n_cand = __builtin_amdgcn_readfirstlane(sh.cand_count[cut_chunk]);
      lds_barrier();
      if (wave == 0) {
        if (lane < cut_chunk) front += cnt;
        if (lane != cut_chunk) cnt = 0;
        leave_chunk_counts(front, cnt, p.n_chunks, sh);
        leave_runs(lane * p.chunk_tokens + front, cnt, p.n_chunks, sh.cand_runs);
      }
      lds_barrier();
    }
  }
  const bool dense = !ALL && n_cand > kCandSlots * HT;                 // uniform; then the registers hold no candidate
  const int n_groups = __builtin_amdgcn_readfirstlane(sh.n_groups);
  if (!ALL && wave == 0) {                                             // the entries of the groups beyond the registers
    const int front = lane < p.n_chunks ? sh.front[lane] : 0;
    const int here = lane < p.n_chunks ? min(front, max(0, SLOTS * HW - sh.group_start[lane]) * kWave) : 0;
    leave_runs(lane * p.chunk_tokens + here, front - here, p.n_chunks, sh.front_runs[0]);
  }
  // group g of the entries in front of the bin
  auto group_at = [&](int g) {
    const int c = chunk_of(sh.group_start, g), first = (g - sh.group_start[c]) * kWave;
    return make_int2(c * p.chunk_tokens + first, min(kWave, sh.front[c] - first));
  };
  auto cand_at = [&](int idx) {
    const int c = chunk_of(sh.cand_start, idx);
    return c * p.chunk_tokens + sh.front[c] + idx - sh.cand_start[c];
  };
  static_assert(SLOTS * HW <= kMaxGroups && kMaxGroups == HT, "at most one group per thread");
  sh.group[tid] = tid < n_groups ? group_at(tid) : make_int2(0, 0);
  uint32_t ckey[kCandSlots], ceps[kCandSlots], key[SLOTS + kCandSlots];
  int cpos[kCandSlots];
  {
    int at[kCandSlots];
#pragma unroll
    for (int i = 0; i < kCandSlots; ++i) at[i] = n_cand > 0 ? cand_at(min(tid + i * HT, n_cand - 1)) : 0;
#pragma unroll
    for (int i = 0; i < kCandSlots; ++i) { ckey[i] = bkey[at[i]]; cpos[i] = bpos[at[i]]; ceps[i] = beps[at[i]]; }
  }
  lds_barrier();
  // Slot i of wave w: group w + HW i
#pragma unroll
  for (int i = 0; i < SLOTS; ++i) {
    const int2 g = sh.group[wave + HW * i];
    key[i] = beps[g.x + min(lane, max(g.y - 1, 0))];
  }
#pragma unroll
  for (int i = 0; i < SLOTS; ++i)
    if (lane >= sh.group[wave + HW * i].y) key[i] = 0u;
#pragma unroll
  for (int i = 0; i < kCandSlots; ++i)
    if (dense || tid + i * HT >= n_cand) ckey[i] = 0u;
  if (tid == 0) { sh.center[0] = ckey[0]; sh.center[1] = n_front > 0 ? key[0] : ceps[0]; }
  lds_barrier();
  const uint32_t center0 = sh.center[0], center1 = sh.center[1];
  // Step 1: the pool is the n_pool tokens of highest score
  Cut top = {least, p.n_pool - n_front, all_candidates};
  if (!plateau) {                                      // uniform
    if (n_cand > kRankCap && !dense) leave_sample(ckey, center0, sh);
    top = list_select<true>(ckey, [&](auto f) {
      if (dense) walk_runs<4>(sh.cand_runs, sh.run_group, p.n_chunks, 0, p.n_chunks, keys_at, [&](u32x4 x, int e) { f(x[e]); });
    }, n_cand, p.n_pool - n_front, center0, dense, least, most - least, sh);
  }
  leave_sample(key, center1, sh);                      // before the candidates join: one barrier less
  HeadCut cut;
  cut.top_thr = top.thr;
  cut.top_tok = kRouteMaxSeqLen;
  if (!top.all_equal) {                                // uniform
    const int first = plateau ? cut_chunk * p.chunk_tokens : 0;
    cut.top_tok = token_cut([&](int a, int b, auto f) {
#pragma unroll
      for (int i = 0; i < kCandSlots; ++i) f(ckey[i], cpos[i]);        // no key is 0
      if (dense)
        walk_runs<2>(sh.cand_runs, sh.run_group, p.n_chunks, a / p.chunk_tokens, b / p.chunk_tokens + 1,
                           [&](int at) { return Tokens{load_entries(bkey, at), load_entries(bpos, at)}; },
                           [&](const Tokens& x, int e) { f(x.key[e], (int)x.tok[e]); });
    }, top.thr, top.quota, first, plateau ? min(n, first + p.chunk_tokens) - 1 : n - 1, sh);
  }
  // Step 3: inside the pool, the n_approx tokens of lowest residual lose their value
#pragma unroll
  for (int i = 0; i < kCandSlots; ++i) key[SLOTS + i] = ckey[i] != 0u && cut.in_pool(ckey[i], cpos[i]) ? ceps[i] : 0u;
  // every pool member of chunks [c0, c1) beyond the registers, or (every) all of them: f(residual key, token)
  auto pool_members = [&](bool every, int c0, int c1, auto f) {
    if (!ALL || every)
      walk_runs<2>(sh.front_runs[every], sh.run_group, p.n_chunks, c0, c1,
                   [&](int at) { return Tokens{load_entries(beps, at), load_entries(bpos, at)}; },
                   [&](const Tokens& x, int e) { f(x.key[e], (int)x.tok[e]); });
    if (every) {
#pragma unroll
      for (int i = 0; i < kCandSlots; ++i)
        if (key[SLOTS + i] != 0u) f(key[SLOTS + i], cpos[i]);
    }
    if (dense)
      walk_runs<2>(sh.cand_runs, sh.run_group, p.n_chunks, c0, c1,
                         [&](int at) { return Entries{load_entries(bkey, at), load_entries(bpos, at), load_entries(beps, at)}; },
                         [&](const Entries& x, int e) { if (cut.in_pool(x.key[e], (int)x.tok[e])) f(x.eps[e], (int)x.tok[e]); });
  };
  Cut low = {0xffffffffu, 0, true};                    // n_approx = 0: none
  cut.low_tok = kRouteMaxSeqLen;
  if (p.n_approx > 0) {
    low = list_select<false>(key, [&](auto f) { if (!ALL) pool_members(false, 0, p.n_chunks, [&](uint32_t k, int) { f(k); }); }, p.n_pool,
                             p.n_approx, center1, false, 1u, 0xfffffffeu, sh);
    if (!low.all_equal) {
      if (wave == 0) leave_runs(lane * p.chunk_tokens, lane < p.n_chunks ? sh.front[lane] : 0, p.n_chunks, sh.front_runs[1]);
      lds_barrier();
      cut.low_tok = token_cut([&](int a, int b, auto f) { pool_members(true, a / p.chunk_tokens, b / p.chunk_tokens + 1, f); }, low.thr, low.quota,
                              0, n - 1, sh);
    }
  }
  cut.low_thr = low.thr;
  cut.any_approx = p.n_approx > 0;
  // Those in registers by their residuals, or (which of the equal keys?) every one by its token
  cut.pool_before = cut.apx_before = 0;
  const int own_first = own_chunk * p.chunk_tokens;
  if (low.all_equal) {
    const int groups_before = min(sh.group_start[own_chunk], SLOTS * HW);
    int apx = 0;
#pragma unroll
    for (int i = 0; i < SLOTS; ++i)
      if (wave + HW * i < groups_before) apx += __popcll(__ballot(p.n_approx > 0 && key[i] >= low.thr));      // uniform
    if (lane == 0) cut.apx_before += apx;
#pragma unroll
    for (int i = 0; i < kCandSlots; ++i)
      if (key[SLOTS + i] != 0u && cpos[i] < own_first) { ++cut.pool_before; cut.apx_before += cut.is_approx(key[SLOTS + i], 0); }
    if (tid == 0) {                                    // the register slots' share of the pool: whole chunks and one cut off
      int in_slots = 0;
      for (int c = 0; c < own_chunk; ++c) in_slots += min(sh.front[c], max(0, (groups_before - sh.group_start[c]) * kWave));
      cut.pool_before += in_slots;
    }
  }
  if (own_chunk > 0 && (!ALL || !low.all_equal))       // uniform
    pool_members(!low.all_equal, 0, own_chunk, [&](uint32_t k, int tok) {
      if (tok < own_first) { ++cut.pool_before; cut.apx_before += cut.is_approx(k, tok); }
    });
  return cut;
}

template <int SLOTS, bool RAGGED>
__global__ __launch_bounds__(HT) void route_list_kernel(KernelArgs<RouteParams, RAGGED> args) {
  RouteParams p = args.p;
  int part, h;
  xcd_chunk_head(part, h);
  const int launch_head = h;
  take_sequence<RAGGED>(p, h);
  const int n = p.n, begin = part * p.part_tokens, end = min(n, begin + p.part_tokens);
  if (begin >= n) return;
  __shared__ ListShared sh;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), tid = threadIdx.x;
  const float* score = p.score + (size_t)h * n;
  const float* eps = p.eps + (size_t)h * n;
  auto load4 = [&](const float* a, int t0, int stop) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (t0 + 4 <= stop) {
      x = *reinterpret_cast<const f32x4_u*>(a + t0);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t0 + e < stop) x[e] = a[t0 + e];
    }
    return x;
  };
  const int own_chunk = begin / p.chunk_tokens, own_first = own_chunk * p.chunk_tokens;
  // the tokens this thread emits first, and those of the part's chunk that lie before it: requested with the tables
  f32x4 sc, ep, own_sc, own_ep;
  pick_from_tables(p.table + (size_t)h * p.n_chunks * kTableStride, p.n_chunks, p.n_pool, sh, [&]() {
    sc = load4(score, begin + 4 * tid, end);
    ep = load4(eps, begin + 4 * tid, end);
    own_sc = load4(score, own_first + 4 * tid, begin);
    own_ep = load4(eps, own_first + 4 * tid, begin);
  });
  const bool fits = __builtin_amdgcn_readfirstlane(sh.pick[2]) <= kCandSlots * HT && __builtin_amdgcn_readfirstlane(sh.n_groups) <= SLOTS * HW;
  HeadCut cut;
  if (__builtin_expect(fits, 1)) cut = cut_head<SLOTS, true>(p, h, own_chunk, sh);      // uniform
  else cut = cut_head<SLOTS, false>(p, h, own_chunk, sh);
  // Members in front of this part: the chunks before its own, then the own chunk's tokens before it
  int pool_before = cut.pool_before, apx_before = cut.apx_before;
  for (int t = own_first; t < begin; t += kHeadBlock) {
    const int t0 = t + 4 * tid;
    if (t != own_first) { own_sc = load4(score, t0, begin); own_ep = load4(eps, t0, begin); }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool pool = t0 + e < begin && cut.in_pool(float_key(own_sc[e]), t0 + e);
      pool_before += pool;
      apx_before += pool && cut.is_approx(~float_key(own_ep[e]), t0 + e);
    }
  }
  int base_r, base_a;
  {
    const int x = wave_total_of_scan(wave_incl_scan_dpp(pool_before)), y = wave_total_of_scan(wave_incl_scan_dpp(apx_before));
    if (lane == 0) { sh.wsum[1][wave] = x; sh.wsum[2][wave] = y; }
    lds_barrier();
    int total = 0, total_a = 0;
#pragma unroll
    for (int w = 0; w < HW; ++w) { total += sh.wsum[1][w]; total_a += sh.wsum[2][w]; }
    base_a = total_a;
    base_r = total - total_a;
    lds_barrier();                                     // the rows are used again below
  }
  p = params_again<RAGGED, RouteParams>(launch_head);
  const int n_retain = p.n_pool - p.n_approx;
  const EmitTarget target = {p.tier + (size_t)h * n, p.idx_retain + (size_t)h * n_retain, p.idx_approx + (size_t)h * p.n_approx, end, n_retain, p.n_approx};
  for (int t = begin; t < end; t += kHeadBlock) {
    const int t0 = t + 4 * tid;
    uint32_t ret4 = 0u, apx4 = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool pool = t0 + e < end && cut.in_pool(float_key(sc[e]), t0 + e);
      const bool apx = pool && cut.is_approx(~float_key(ep[e]), t0 + e);
      ret4 |= (pool && !apx ? 1u : 0u) << e;
      apx4 |= (apx ? 1u : 0u) << e;
    }
    int at, own;
    head_scan<HT>(__popc(ret4) + (__popc(apx4) << 16), sh.wsum[0], at, own);
    const int own_r = low16(own), own_a = high16(own);
    if (t0 < end) list_tokens(t0, ret4, apx4, low16(at), high16(at), own_r, sh.list);
    if (t + kHeadBlock < end) { sc = load4(score, t0 + kHeadBlock, end); ep = load4(eps, t0 + kHeadBlock, end); }
    lds_barrier();                                     // the list is whole
    if (t0 < end) store_tiers(target, t0, ret4, apx4);
    store_indices<HT>(target, sh.list, own_r, own_a, base_r, base_a);
    if (p.g.k) copy_rows<HT>(p.g, h, p.n_approx, sh.list, own_r, own_a, base_r, base_a);
    base_r += own_r;
    base_a += own_a;
    lds_barrier();                                     // the list may be written again
  }
}

// nothing is kept: every token is evicted
__global__ __launch_bounds__(256) void route_evict_all_kernel(uint8_t* __restrict__ tier, size_t total) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < total) tier[i] = VECTOR_TIER_EVICT;
}

// ---------------------------------------------------------------------------
// compaction: one 16-byte piece per thread, P pieces per row
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void gather_rows_kernel(GatherParams p) {
  const int h = blockIdx.y;
  const int seg = blockIdx.z;                       // seg 0: k_ret, 1: v_ret, 2: k_apx
  const int pieces = p.row_bytes / 16;
  const int rows = (seg == 2) ? p.n_approx : p.n_retain;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int row = (int)(gid / pieces), piece = (int)(gid - (int64_t)row * pieces);
  if (row >= rows) return;
  const int32_t* idx = (seg == 2) ? p.idx_approx + (size_t)h * p.n_approx : p.idx_retain + (size_t)h * p.n_retain;
  int tok = idx[row];
  tok = min(max(tok, 0), p.n - 1);                  // an index list is trusted, but never walk out of the tensor
  const int64_t hs = p.hps ? h / p.hps : 0, hh = p.hps ? h % p.hps : h;      // sequence and KV head of the launch head
  const unsigned char* src = (seg == 1) ? p.v + hs * p.v_sb + hh * p.v_sh + (int64_t)tok * p.v_st
                                        : p.k + hs * p.k_sb + hh * p.k_sh + (int64_t)tok * p.k_st;
  unsigned char* dst = (seg == 0) ? p.k_ret + ((size_t)h * p.cap_retain + row) * p.row_bytes
                     : (seg == 1) ? p.v_ret + ((size_t)h * p.cap_retain + row) * p.row_bytes
                                  : p.k_apx + ((size_t)h * p.n_approx + row) * p.row_bytes;
  *reinterpret_cast<uint4*>(dst + piece * 16) = *reinterpret_cast<const uint4*>(src + piece * 16);
}

}  // namespace

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static int bucket_threads(int chunk_tokens) { return chunk_tokens <= kMinChunk ? 512 : 1024; }
static int route_chunk_tokens(int seq_len) {
  int ch = kMinChunk;
  while ((seq_len + ch - 1) / ch > kMaxChunks) ch *= 2;
  return ch;
}

namespace {
struct RouteLayout {
  int chunk_tokens, n_chunks;
  size_t off_range, off_table, off_bkey, off_bpos, off_beps, total;
};
RouteLayout route_layout(int n_kv_heads, int seq_len) {
  RouteLayout L;
  L.chunk_tokens = route_chunk_tokens(seq_len);
  L.n_chunks = (seq_len + L.chunk_tokens - 1) / L.chunk_tokens;
  const size_t tables = align_up((size_t)n_kv_heads * L.n_chunks * kTableStride * sizeof(uint16_t), 256);
  const size_t per_token = align_up((size_t)n_kv_heads * seq_len * sizeof(uint32_t), 256);
  size_t off = 0;
  L.off_range = off;  off += align_up((size_t)n_kv_heads * route_mass_range_slots(n_kv_heads, seq_len) * sizeof(float4), 256);
  L.off_table = off;  off += tables;
  L.off_bkey = off;   off += per_token;          // behind other arrays: walk_runs reads up to 12 bytes in front of a list
  L.off_bpos = off;   off += per_token;
  L.off_beps = off;   off += per_token;
  L.total = off;
  return L;
}

void fill_bucket_params(BucketParams& bp, const RouteLayout& L, void* route_ws) {
  unsigned char* w8 = reinterpret_cast<unsigned char*>(route_ws);
  bp.table = w8 ? reinterpret_cast<uint16_t*>(w8 + L.off_table) : nullptr;
  bp.bkey = w8 ? reinterpret_cast<uint32_t*>(w8 + L.off_bkey) : nullptr;
  bp.bpos = w8 ? reinterpret_cast<int32_t*>(w8 + L.off_bpos) : nullptr;
  bp.beps = w8 ? reinterpret_cast<uint32_t*>(w8 + L.off_beps) : nullptr;
  bp.range = w8 ? reinterpret_cast<const float4*>(w8 + L.off_range) : nullptr;
  bp.n_range = 0;
  bp.log_ref = 0.f;
  bp.seq_table = nullptr;
  bp.seq_hps = 0;
  bp.chunk_tokens = L.chunk_tokens;
  bp.n_chunks = L.n_chunks;
}
}  // namespace

size_t route_workspace_bytes(int n_kv_heads, int seq_len) { return route_layout(n_kv_heads, seq_len).total; }

// the scorer's second pass has at most 1024 workgroups, of no fewer than 32 tokens
int route_mass_range_slots(int n_kv_heads, int seq_len) {
  const int most = n_kv_heads < 1024 ? 1024 / n_kv_heads : 1;
  return (seq_len + 31) / 32 < most ? (seq_len + 31) / 32 : most;
}
void* route_mass_range(void* route_ws, int n_kv_heads) {
  return reinterpret_cast<unsigned char*>(route_ws) + route_layout(n_kv_heads, 1).off_range;
}

namespace {
BucketParams pool_bucket_params(const float* mass, float* score, const float* eps, int n_kv_heads, int seq_len, int n_prefix, int pool_kernel,
                                int pool_mode, void* route_ws, int n_range, RouteLayout& L) {
  L = route_layout(n_kv_heads, seq_len);
  BucketParams bp;
  bp.src = mass; bp.score = score; bp.eps = eps; bp.n = seq_len; bp.n_prefix = n_prefix; bp.kernel = pool_kernel; bp.inv_kernel = 1.0f / (float)pool_kernel; bp.take_max = pool_mode == VECTOR_POOL_MAX;
  fill_bucket_params(bp, L, route_ws);
  bp.n_range = route_ws ? n_range : 0;
  bp.log_ref = -log2f((float)(n_prefix > 0 ? n_prefix : 1));     // as in the scorer's second pass
  return bp;
}

RouteParams route_params(int n_kv_heads, int all_heads, int seq_len, const float* score, const float* eps, int n_pool, int n_approx, uint8_t* tier,
                         int32_t* idx_retain, int32_t* idx_approx, void* ws) {
  const RouteLayout L = route_layout(n_kv_heads, seq_len);
  unsigned char* w8 = reinterpret_cast<unsigned char*>(ws);
  RouteParams p;
  p.score = score; p.eps = eps; p.n = seq_len; p.n_pool = n_pool; p.n_approx = n_approx;
  p.chunk_tokens = L.chunk_tokens; p.n_chunks = L.n_chunks;
  // one workgroup per CU: finding the thresholds costs each the same, whatever its part
  const int parts = all_heads >= 256 ? 1 : 256 / all_heads;
  p.part_tokens = (int)(((int64_t)(seq_len + parts - 1) / parts + 63) / 64 * 64);
  p.table = reinterpret_cast<const uint16_t*>(w8 + L.off_table);
  p.bkey = reinterpret_cast<const uint32_t*>(w8 + L.off_bkey);
  p.bpos = reinterpret_cast<const int32_t*>(w8 + L.off_bpos);
  p.beps = reinterpret_cast<const uint32_t*>(w8 + L.off_beps);
  p.tier = tier; p.idx_retain = idx_retain; p.idx_approx = idx_approx;
  p.g = GatherParams{};
  p.seq_table = nullptr; p.seq_hps = 0;
  return p;
}
// the fewest register slots that hold the pool: its groups of 64, a last one that is not full per chunk, over the waves
template <bool RAGGED> void (*list_kernel(int n_pool, int n_chunks))(KernelArgs<RouteParams, RAGGED>) {
  const int groups = n_pool / kWave + n_chunks;
  if (groups <= 8 * HW) return route_list_kernel<8, RAGGED>;
  if (groups <= 16 * HW) return route_list_kernel<16, RAGGED>;
  return route_list_kernel<32, RAGGED>;
}
unsigned route_parts(const RouteParams& p) { return (unsigned)((p.n + p.part_tokens - 1) / p.part_tokens); }

unsigned gather_grid_x(const GatherParams& p) {
  const int pieces = p.row_bytes / 16;
  const int max_rows = p.n_retain > p.n_approx ? p.n_retain : p.n_approx;
  return (unsigned)(((int64_t)max_rows * pieces + 255) / 256);
}
}  // namespace

int launch_pool_scores(const float* mass, float* score, const float* eps, int n_kv_heads, int seq_len, int n_prefix, int pool_kernel, int pool_mode,
                       void* route_ws, int n_range, hipStream_t stream) {
  if (n_range < 0 || n_range > route_mass_range_slots(n_kv_heads, seq_len) || (route_ws && !eps)) return VECTOR_ERR_ARG;
  RouteLayout L;
  const BucketParams bp = pool_bucket_params(mass, score, eps, n_kv_heads, seq_len, n_prefix, pool_kernel, pool_mode, route_ws, n_range, L);
  const auto kernel = L.chunk_tokens <= kMinChunk ? route_bucket_kernel<512, true, false> : route_bucket_kernel<1024, true, false>;
  VEC_LAUNCH(K_POOL, kernel, dim3(L.n_chunks, n_kv_heads), dim3(bucket_threads(L.chunk_tokens)), 0, stream, KernelArgs<BucketParams, false>{bp});
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

int launch_route(int n_kv_heads, int seq_len, const float* score, const float* eps, int n_pool, int n_approx, uint8_t* tier,
                 int32_t* idx_retain, int32_t* idx_approx, void* ws, bool have_buckets, const PackedRows* rows, hipStream_t stream) {
  if (n_approx < 0 || n_pool < n_approx || n_pool > seq_len) return VECTOR_ERR_ARG;      // the selections rely on it
  if (n_pool == 0) {
    const size_t total = (size_t)n_kv_heads * seq_len;
    VEC_LAUNCH(K_ROUTE, route_evict_all_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream, tier, total);
    VEC_HIP(hipGetLastError());
    return VECTOR_OK;
  }
  if (!have_buckets && route_head_fits(seq_len))
    return launch_route_head(n_kv_heads, seq_len, score, eps, n_pool, n_approx, tier, idx_retain, idx_approx, nullptr, rows, stream);
  RouteParams p = route_params(n_kv_heads, n_kv_heads, seq_len, score, eps, n_pool, n_approx, tier, idx_retain, idx_approx, ws);
  if (rows)
    p.g = gather_params(*rows->shape, rows->k, rows->v, idx_retain, idx_approx, n_pool - n_approx, n_approx, rows->k_ret, rows->v_ret,
                        rows->k_apx, rows->cap_retain, rows->stack);
  const bool t_ = timing_enabled();
  if (t_) timing_begin(K_ROUTE, stream);             // the launches count as one routing step
  if (!have_buckets) {
    const RouteLayout L = route_layout(n_kv_heads, seq_len);
    BucketParams bp;
    bp.src = score; bp.score = nullptr; bp.eps = eps; bp.n = seq_len; bp.n_prefix = seq_len; bp.kernel = 1; bp.inv_kernel = 1.f; bp.take_max = 0;
    fill_bucket_params(bp, L, ws);
    const auto kernel = L.chunk_tokens <= kMinChunk ? route_bucket_kernel<512, false, false> : route_bucket_kernel<1024, false, false>;
    hipLaunchKernelGGL(kernel, dim3(L.n_chunks, n_kv_heads), dim3(bucket_threads(L.chunk_tokens)), 0, stream, KernelArgs<BucketParams, false>{bp});
  }
  hipLaunchKernelGGL(list_kernel<false>(n_pool, p.n_chunks), dim3(route_parts(p), n_kv_heads), dim3(HT), 0, stream, KernelArgs<RouteParams, false>{p});
  if (t_) timing_end(K_ROUTE, stream);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

int launch_compact(const vector_shape& s, const void* k, const void* v, const int32_t* idx_retain,
                   const int32_t* idx_approx, int n_retain, int n_approx, void* k_ret, void* v_ret, void* k_apx,
                   int cap_retain, hipStream_t stream, const SeqStack* stack) {
  const GatherParams p = gather_params(s, k, v, idx_retain, idx_approx, n_retain, n_approx, k_ret, v_ret, k_apx, cap_retain, stack);
  const unsigned gx = gather_grid_x(p);
  if (gx == 0) return VECTOR_OK;
  VEC_LAUNCH(K_GATHER, gather_rows_kernel, dim3(gx, s.n_kv_heads, 3), dim3(256), 0, stream, p);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

// ---------------------------------------------------------------------------
// several sequences of different lengths in one set of launches
// ---------------------------------------------------------------------------
size_t route_ragged_table_bytes(int count) {
  return align_up(sizeof(BucketParams) * count, 256) + align_up(sizeof(RouteParams) * count, 256);
}

int launch_pool_scores_ragged(const PoolSeq* seqs, int count, int n_kv_heads, int pool_kernel, int pool_mode, void* tables,
                              hipStream_t stream) {
  if (count < 1 || count > kMaxRaggedSeqs) return VECTOR_ERR_ARG;
  BucketParams host[kMaxRaggedSeqs];
  unsigned gx = 0;
  int longest_chunk = 0;
  for (int b = 0; b < count; ++b) {
    if (!seqs[b].route_ws || !seqs[b].eps || seqs[b].n_range < 0 || seqs[b].n_range > route_mass_range_slots(n_kv_heads, seqs[b].seq_len)) return VECTOR_ERR_ARG;
    RouteLayout L;
    host[b] = pool_bucket_params(seqs[b].mass, seqs[b].score, seqs[b].eps, n_kv_heads, seqs[b].seq_len, seqs[b].n_prefix, pool_kernel, pool_mode,
                                 seqs[b].route_ws, seqs[b].n_range, L);
    if ((unsigned)L.n_chunks > gx) gx = (unsigned)L.n_chunks;
    longest_chunk = std::max(longest_chunk, L.chunk_tokens);
  }
  KernelArgs<BucketParams, true> args;
  const int rc = ragged_args(host, count, n_kv_heads, tables, stream, args);
  if (rc != VECTOR_OK) return rc;
  const auto kernel = longest_chunk <= kMinChunk ? route_bucket_kernel<512, true, true> : route_bucket_kernel<1024, true, true>;
  VEC_LAUNCH(K_POOL, kernel, dim3(gx, (unsigned)count * n_kv_heads), dim3(bucket_threads(longest_chunk)), 0, stream, args);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

int launch_route_compact_ragged(const vector_shape& s, const RaggedSeq* seqs, int count, void* tables, hipStream_t stream) {
  if (count < 1 || count > kMaxRaggedSeqs) return VECTOR_ERR_ARG;
  RouteParams host[kMaxRaggedSeqs];
  unsigned parts = 0;
  int most_pool = 0, most_chunks = 0;
  for (int b = 0; b < count; ++b) {
    const RaggedSeq& q = seqs[b];
    // the selections rely on it; nothing kept: that sequence goes through launch_route on its own
    if (q.n_pool < 1 || q.n_approx < 0 || q.n_pool < q.n_approx || q.n_pool > q.shape.seq_len) return VECTOR_ERR_ARG;
    host[b] = route_params(s.n_kv_heads, count * s.n_kv_heads, q.shape.seq_len, q.score, q.eps, q.n_pool, q.n_approx, q.tier, q.idx_retain,
                           q.idx_approx, q.route_ws);
    host[b].g = gather_params(q.shape, q.k, q.v, q.idx_retain, q.idx_approx, q.n_pool - q.n_approx, q.n_approx, q.k_ret, q.v_ret, q.k_apx,
                              q.cap_retain, nullptr);
    parts = std::max(parts, route_parts(host[b]));
    most_pool = std::max(most_pool, q.n_pool);
    most_chunks = std::max(most_chunks, host[b].n_chunks);
  }
  unsigned char* t8 = reinterpret_cast<unsigned char*>(tables) + align_up(sizeof(BucketParams) * count, 256);
  KernelArgs<RouteParams, true> args;
  const int rc = ragged_args(host, count, s.n_kv_heads, t8, stream, args);
  if (rc != VECTOR_OK) return rc;
  VEC_LAUNCH(K_ROUTE, list_kernel<true>(most_pool, most_chunks), dim3(parts, (unsigned)count * s.n_kv_heads), dim3(HT), 0, stream, args);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

// ---------------------------------------------------------------------------
// parameter tables: host bytes to device memory as the arguments of small copy launches
// ---------------------------------------------------------------------------
namespace {
constexpr int kBlobBytes = 3584;
struct Blob { uint4 w[kBlobBytes / 16]; };
__global__ __launch_bounds__(256) void table_copy_kernel(Blob blob, uint4* dst, int words) {
  for (int i = threadIdx.x; i < words; i += 256) dst[i] = blob.w[i];
}
}  // namespace

int upload_table(const void* host, size_t bytes, void* dev, hipStream_t stream) {
  if (!host || !dev || (reinterpret_cast<uintptr_t>(dev) & 15u)) return VECTOR_ERR_ARG;
  const unsigned char* src = reinterpret_cast<const unsigned char*>(host);
  unsigned char* dst = reinterpret_cast<unsigned char*>(dev);
  for (size_t off = 0; off < bytes; off += kBlobBytes) {
    const size_t part = bytes - off < (size_t)kBlobBytes ? bytes - off : (size_t)kBlobBytes;
    Blob blob;
    memset(&blob, 0, sizeof(blob));
    memcpy(&blob, src + off, part);
    hipLaunchKernelGGL(table_copy_kernel, dim3(1), dim3(256), 0, stream, blob, reinterpret_cast<uint4*>(dst + off), (int)((part + 15) / 16));
  }
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

}  // namespace vec
