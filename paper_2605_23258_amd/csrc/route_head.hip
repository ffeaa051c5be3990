// Routing of a whole head in one launch (Section 3.2, Steps 1 and 3, and the packed cache), for heads of
// up to 16384 tokens: pooling of the attention mass, both selections, tiers, index lists and
// row copies.
//
// The chain of selections is latency: with the pieces of a head spread over workgroups, every exchange
// between them is a kernel boundary, and a boundary costs 4 us or more whatever the size.  So nothing is exchanged.
// Every workgroup of a head loads the head's scores and residuals whole into registers (16384 tokens: 16 + 16 per
// thread) and finds both thresholds itself; then it emits and copies its own part of the tokens.  The redundant
// part is about 50 vector instructions and two LDS atomics per token and workgroup.  At 8192 tokens x 8 heads 13.1 us from the first
// workgroup's start to the last one's end (a kernel trace has 15), 12 in the mean workgroup (loads 1.6, pooling 1.2, selections
// 3.4 and 2.8, list 1.4, rows 2); at 12289 tokens with a maximum pooled 18.6 (19.4).
//
// The line to the two launches of route_compact.hip.  A whole compression pass in us, bf16, d = 128, 64 query rows,
// this launch (with 24576 tokens in registers for the last two lengths) against the two:
//     heads    2049        8192        14337       16384       20011       24576 tokens
//       1   24 /  35    29 /  37    38 /  42    38 /  42    42 /  42    42 /  42
//       8   25 /  35    32 /  41    43 /  48    44 /  49    59 /  57    64 /  63
//      64   42 /  52   104 / 118   185 / 195   200 / 211   263 / 276   312 / 325
// Up to 16384 tokens this launch is the faster one for any number of heads.  Beyond, for up to 16 heads, it is not; for many
// more it still would be by 3 to 5 %, which is not used: registers for 24576 tokens would be one more set of kernels.
//
// A selection finds the k-th largest of the keys in registers: one LDS histogram over buckets laid
// where a sample says that the keys lie (DigitMap), then the keys of the bucket that holds it are ranked
// against each other by (key, lower token first); a bucket of more keys than kRankCap is cut further over the
// range its keys really take (narrow()), and equal keys by histograms over their tokens.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "plan.hpp"
#include "route_common.hpp"

namespace vec {

namespace {

constexpr int kMaxHead = 16384;                 // tokens
// Half of the widest pooling kernel: two quads on either side of a token's own.  Wider ones are pooled by a launch of their own,
// and unequal prompts routed by two more.  Kernel 13 with that limit at nine, and now, us a compression pass: 8192 tokens, 8 heads
// 38.6 / 34.1, 2049 30.5 / 25.8, five prompts of 1500 to 6000 tokens 80.8 / 56.1, two of 750 and 1500, two heads 42 / 25.
constexpr int kMaxHalf = 8;
constexpr int kUnit = 4 * kWave;                // tokens of a wave in a block: what the head is shared out in

struct HeadParams {
  const float* src;       // POOL: attention mass [H, n]; otherwise the scores [H, n]
  float* score;           // POOL: output [H, n]
  const float* eps;       // [H, n]
  int n, n_prefix, half, take_max;      // POOL: prefix columns, half the kernel (at most kMaxHalf), maximum instead of mean
  float inv_kernel;       // of the kernel
  int n_pool, n_approx;
  int units_per_part;     // units of kUnit tokens that a workgroup emits
  int parts;              // workgroups per head
  uint8_t* tier; int32_t* idx_retain; int32_t* idx_approx;
  GatherParams g;         // row copies (k null: none)
  const HeadParams* seq_table;          // RAGGED launches: the sequences' parameter blocks, seq_hps heads each
  int seq_hps;
};

template <int NT> struct HeadShared {
  __align__(16) int hist[kHeadBins];
  __align__(16) f32x4 first[2][kMaxHead / kUnit], last[2][kMaxHead / kUnit];     // POOL: the quads at the edges of every wave's run of a block, and the next ones
  __align__(16) unsigned long long cand[kRankCap];     // (key, ~token)
  __align__(16) int list[kBlock<NT>];                  // tokens whose rows this workgroup copies: retained, then approximated
  int wsum[3][kWaves<NT>];
  float stat[3][kWaves<NT>];
  uint32_t range[2][kWaves<NT>];
  uint32_t center[2];
  int pick[3];            // bucket, #keys above it, keys in it
  int n_cand;
  uint32_t thr, thr_tok, next_key;
};

// the k-th largest (key, lower token first): keys above thr, and keys equal to thr up to token tok, are the k;
// all_equal: every key equal to thr is among them
struct Threshold { uint32_t thr, tok; bool all_equal; };

// token of a thread's slot; base: first_token(), taken anew where slots are walked (its sums with the slots'
// constants would otherwise be kept in registers for the whole kernel)
__device__ __forceinline__ int first_token() {
  int t = (int)threadIdx.x * 4;
  asm volatile("" : "+v"(t));
  return t;
}
template <int NT> __device__ __forceinline__ int head_token(int base, int slot) { return (slot >> 2) * kBlock<NT> + base + (slot & 3); }

// Threshold of the k largest of the workgroup's keys (0: no key in that slot); 1 <= k <= number of keys.
// center: a typical key.  Starts by clearing the histogram; the caller has passed a barrier since the
// last use of sh.
template <int NT, int NS>
__device__ __forceinline__ Threshold head_select(const uint32_t (&key)[NS], int k, uint32_t center, HeadShared<NT>& sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  clear_bins<NT>(sh.hist);
  // mean and deviation of a sample (in units of 4096 keys, about the center): where to lay the buckets
  float cnt = 0.f, s1 = 0.f, s2 = 0.f;
  constexpr int kStep = NS / 4 > 8 ? 2 : 1;
#pragma unroll
  for (int j = 0; j < NS / 4; j += kStep) {
    const uint32_t x = key[4 * j];
    const bool ok = x > 0x007fffffu && x < 0xff800000u;                 // a finite number
    const float dlt = ok ? (float)((int)(x >> 12) - (int)(center >> 12)) : 0.f;
    cnt += ok ? 1.f : 0.f;
    s1 += dlt;
    s2 = fmaf(dlt, dlt, s2);
  }
  cnt = wave_sum_dpp(cnt); s1 = wave_sum_dpp(s1); s2 = wave_sum_dpp(s2);
  if (lane == 0) { sh.stat[0][wave] = cnt; sh.stat[1][wave] = s1; sh.stat[2][wave] = s2; }
  lds_barrier();
  if (threadIdx.x == 0) { sh.n_cand = 0; sh.next_key = 0u; }
  cnt = sum_of_waves<NT>(sh.stat[0], lane); s1 = sum_of_waves<NT>(sh.stat[1], lane); s2 = sum_of_waves<NT>(sh.stat[2], lane);
  auto each = [&](auto f) {
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      f(key[i]);
      if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);              // four at a time: the digits of all would not fit the registers
    }
  };
  uint32_t lo, span;
  int count;
  if (!(cnt >= 32.f && s2 == 0.f && around_center<NT>(each, center, lo, span, k, count, sh.wsum[0]))) {      // uniform
    const DigitMap map = digit_map_about(center, cnt, s1, s2);
    each([&](uint32_t x) { if (x != 0u) atomicAdd(&sh.hist[map.digit(x)], 1); });
    lds_barrier();
    int d, above;
    pick_bin<NT>(sh.hist, sh.wsum[0], sh.pick, k, d, above, count);
    k -= above;
    bucket_range(map, d, lo, span);
  }
  narrow<NT>(each, false, lo, span, k, count, sh.hist, sh.wsum[0], sh.pick, sh.range);
  Threshold out;
  if (count > kRankCap) {
    // one key, many tokens: cut the range of last - token the same way until one is left
    const uint32_t thr = lo;
    constexpr uint32_t kLast = NS * NT - 1;
    uint32_t tlo = 0u, tspan = k == count ? 0u : kLast;                 // uniform; all of them taken: no cut
    out.all_equal = tspan == 0u;
    while (tspan != 0u) {
      const int s = max(0, 21 - (int)__clz(tspan));
      clear_bins<NT>(sh.hist);
      lds_barrier();
      const int base = first_token();
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const uint32_t v = kLast - (uint32_t)head_token<NT>(base, i) - tlo;
        if (key[i] == thr && v <= tspan) atomicAdd(&sh.hist[v >> s], 1);
        __builtin_amdgcn_sched_barrier(0);
      }
      lds_barrier();
      int d, above;
      pick_bin<NT>(sh.hist, sh.wsum[0], sh.pick, k, d, above, count);
      k -= above;
      tlo += (uint32_t)d << s;
      tspan = min(tspan - ((uint32_t)d << s), (1u << s) - 1u);
    }
    out.thr = thr; out.tok = kLast - tlo;
    lds_barrier();
    return out;
  }
  const int base = first_token();
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    if (key[i] - lo <= span) {
      const int at = atomicAdd(&sh.n_cand, 1);
      if (at < kRankCap) sh.cand[at] = ((unsigned long long)key[i] << 32) | (uint32_t)~head_token<NT>(base, i);
    }
    if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
  }
  lds_barrier();
  if ((int)threadIdx.x < count) {
    const unsigned long long mine = sh.cand[threadIdx.x];
    int rank = 0;
#pragma unroll 4
    for (int j = 0; j < count; ++j) rank += sh.cand[j] > mine;
    if (rank == k - 1) { sh.thr = (uint32_t)(mine >> 32); sh.thr_tok = ~(uint32_t)mine; }
    if (rank == k) sh.next_key = (uint32_t)(mine >> 32);
  }
  lds_barrier();
  out.thr = sh.thr; out.tok = sh.thr_tok; out.all_equal = sh.next_key != sh.thr;
  return out;
}

// NT threads; J: blocks of 4 NT tokens a head may have
template <int NT, int J, bool POOL, bool RAGGED>
__global__ __launch_bounds__(NT) void route_head_kernel(RunArgs<HeadParams, RAGGED> args) {
  HeadParams p = args.p;
  int part, h, launch_head = 0;
  if constexpr (RAGGED) {
    const int hps = p.seq_hps;
    int seq;
    const int r = take_workgroup<RunArgs<HeadParams, true>>(p, seq);
    h = r / p.parts;
    part = r - h * p.parts;
    launch_head = seq * hps + h;
  } else {
    xcd_chunk_head(part, h);
  }
  const int n = p.n;
  constexpr int NW = kWaves<NT>;
  const int n_units = (n + kUnit - 1) / kUnit;
  const int unit0 = part * p.units_per_part, unit1 = min(n_units, unit0 + p.units_per_part);      // what this workgroup emits
  __shared__ HeadShared<NT> sh;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

  const float* src = p.src + (size_t)h * n;
  const float* eps = p.eps + (size_t)h * n;
  auto load4 = [&](const float* a, int t0) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (t0 + 4 <= n) {
      x = *reinterpret_cast<const f32x4_u*>(a + t0);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t0 + e < n) x[e] = a[t0 + e];
    }
    return x;
  };
  f32x4 q[J], ev[J];
#pragma unroll
  for (int j = 0; j < J; ++j) q[j] = load4(src, j * kBlock<NT> + (int)threadIdx.x * 4);
#pragma unroll
  for (int j = 0; j < J; ++j) ev[j] = load4(eps, j * kBlock<NT> + (int)threadIdx.x * 4);

  uint32_t key[J * 4];
  // a typical token, for the samples: the middle of the first block (or of what there is of it)
  const bool center_thread = (int)threadIdx.x == min(n, kBlock<NT>) / 8;
  if constexpr (POOL) {
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int t0 = j * kBlock<NT> + (int)threadIdx.x * 4;
      if (t0 - lane * 4 + 4 * kWave > p.n_prefix) {            // uniform per wave: window columns have no mass
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (t0 + e >= p.n_prefix) q[j][e] = 0.f;
      }
      if (lane < 2) sh.first[lane][j * NW + wave] = q[j];
      if (lane > 61) sh.last[63 - lane][j * NW + wave] = q[j];
    }
    lds_barrier();
    float* dst = p.score + (size_t)h * n;
    // One block after the other through `fold`, which makes the pooled value of token e out of the masses around its quad: those of
    // one or two quads on either side.
    auto pool_blocks = [&](auto quads, auto fold) __attribute__((always_inline)) {
      constexpr int Q = decltype(quads)::value;
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int t0 = j * kBlock<NT> + (int)threadIdx.x * 4, slot = j * NW + wave;
        float m[4 * (2 * Q + 1)];
#pragma unroll
        for (int e = 0; e < 4; ++e) m[4 * Q + e] = q[j][e];
#pragma unroll
        for (int d = 1; d <= Q; ++d) {
          f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
          if (slot > 0) lo = sh.last[d - 1][slot - 1];
          if (slot + 1 < J * NW) hi = sh.first[d - 1][slot + 1];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            m[4 * (Q - d) + e] = dpp_take_f<0x138, 0xf>(lo[e], m[4 * (Q - d + 1) + e]);         // wave_shr:1, the quad before
            m[4 * (Q + d) + e] = dpp_take_f<0x130, 0xf>(hi[e], m[4 * (Q + d - 1) + e]);         // wave_shl:1, the quad after
          }
        }
        f32x4 s;
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] = fold(m + 4 * Q + e);
        if (t0 - lane * 4 + 4 * kWave > p.n_prefix) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (t0 + e >= p.n_prefix) s[e] = INFINITY;
        }
        if (slot >= unit0 && slot < unit1) {
          if (t0 + 4 <= n) {
            *reinterpret_cast<f32x4_u*>(dst + t0) = s;
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (t0 + e < n) dst[t0 + e] = s[e];
          }
        }
        q[j] = s;
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // In ascending token order; mass is never negative.  Half the kernel is a constant of the code: as a number to compare with,
    // the maximum over 7 took 0.9 us longer at 12289 tokens.  The mean over 7 comes first: code that is jumped to is code that
    // has to be waited for (0.1 us).
    auto mean_over = [&](auto half) __attribute__((always_inline)) {
      constexpr int H = decltype(half)::value;
      pool_blocks(std::integral_constant<int, (H > 4 ? 2 : 1)>{}, [&](const float* m) __attribute__((always_inline)) {
        float acc = m[-H];
#pragma unroll
        for (int dlt = 1 - H; dlt <= H; ++dlt) acc += m[dlt];
        return pool_mean(acc, (float)(2 * H + 1), p.inv_kernel);
      });
    };
    auto pool_with = [&](auto half) __attribute__((always_inline)) {
      constexpr int H = decltype(half)::value;
      if (p.take_max) {
        pool_blocks(std::integral_constant<int, (H > 4 ? 2 : 1)>{}, [&](const float* m) __attribute__((always_inline)) {
          float most = 0.f;
#pragma unroll
          for (int dlt = -H; dlt <= H; ++dlt) most = fmaxf(most, m[dlt]);
          return most;
        });
      } else {
        mean_over(half);
      }
    };
    if (__builtin_expect(p.half == 3 && !p.take_max, 1)) {       // uniform
      mean_over(std::integral_constant<int, 3>{});
    } else {
      switch (p.half) {
        case 0: pool_with(std::integral_constant<int, 0>{}); break;
        case 1: pool_with(std::integral_constant<int, 1>{}); break;
        case 2: pool_with(std::integral_constant<int, 2>{}); break;
        case 3: pool_with(std::integral_constant<int, 3>{}); break;
        case 4: pool_with(std::integral_constant<int, 4>{}); break;
        case 5: pool_with(std::integral_constant<int, 5>{}); break;
        case 6: pool_with(std::integral_constant<int, 6>{}); break;
        case 7: pool_with(std::integral_constant<int, 7>{}); break;
        default: pool_with(std::integral_constant<int, kMaxHalf>{}); break;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) key[4 * j + e] = float_key(q[j][e]);
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int t0 = j * kBlock<NT> + (int)threadIdx.x * 4;
    if (t0 - lane * 4 + 4 * kWave > n) {                       // no key beyond the head's end
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t0 + e >= n) key[4 * j + e] = 0u;
    }
  }
  if (center_thread) { sh.center[0] = key[0]; sh.center[1] = ~float_key(ev[0][0]); }
  lds_barrier();
  const uint32_t center0 = sh.center[0], center1 = sh.center[1];

  // Step 1: the pool.  Then key[] turns into the residual keys of its members (smaller residual, larger
  // key), 0 elsewhere, and Step 3: the n_approx tokens of lowest residual in it lose their value.  One
  // copy of the selection's code for both: the instruction cache is filled once.
  static_assert(4 * J <= 32, "a bit per slot");
  uint32_t in_pool = 0, in_apx = 0;                            // bit i: slot i
#pragma unroll 1
  for (int step = 0; step < 2; ++step) {
    const int k = step == 0 ? p.n_pool : p.n_approx;
    if (k == 0) break;
    const Threshold t = head_select(key, k, step == 0 ? center0 : center1, sh);
    uint32_t bits = 0u;
    const int base = first_token();
#pragma unroll
    for (int i = 4 * J - 1; i >= 0; --i) {                     // shifting in from the last slot: compare and add-with-carry
      const bool in = key[i] >= t.thr;
      bits = bits + bits + (in ? 1u : 0u);
      if ((i & 3) == 0) __builtin_amdgcn_sched_barrier(0);
    }
    if (!t.all_equal) {                                        // uniform: some keys equal to the threshold stay out
#pragma unroll
      for (int i = 0; i < 4 * J; ++i)
        if (key[i] == t.thr && (uint32_t)head_token<NT>(base, i) > t.tok) bits &= ~(1u << i);
    }
    if (step == 1) { in_apx = bits; break; }
    in_pool = bits;
#pragma unroll
    for (int i = 0; i < 4 * J; ++i) {
      key[i] = (bits >> i) & 1u ? ~float_key(ev[i >> 2][i & 3]) : 0u;
      if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
  }
  const uint32_t in_ret = in_pool & ~in_apx;
  // fewer tokens leave the registers for them (1024 tokens: the second read costs 0.4 us; 8192 and 12289 gain 0.6 and 1.4)
  if constexpr (J * NT >= 2048) p = params_again<RAGGED, HeadParams>(launch_head);
  // ranks: members in earlier blocks, then those of the waves before, then the exclusive prefix inside the wave
  const int block0 = unit0 / NW, block1 = (unit1 - 1) / NW + 1;
  const uint32_t earlier_slots = (1u << (4 * block0)) - 1u;          // block0 < J
  const int earlier = wave_incl_scan_dpp(__popc(in_ret & earlier_slots) + (__popc(in_apx & earlier_slots) << 16));
  if (lane == 63) sh.wsum[1][wave] = earlier;
  int carry = 0;
  const int n_retain = p.n_pool - p.n_approx;
  const EmitTarget target = {p.tier + (size_t)h * n, p.idx_retain + (size_t)h * n_retain, p.idx_approx + (size_t)h * p.n_approx, n, n_retain, p.n_approx};
  for (int b = block0; b < block1; ++b) {
    const int wave0 = max(unit0 - b * NW, 0), wave1 = min(unit1 - b * NW, NW);
    const uint32_t ret4 = (in_ret >> (4 * b)) & 15u, apx4 = (in_apx >> (4 * b)) & 15u;
    const int mine = __popc(ret4) + (__popc(apx4) << 16), incl = wave_incl_scan_dpp(mine);
    if (lane == 63) sh.wsum[2][wave] = incl;
    lds_barrier();
    const int x = row_incl_scan<NT>(sh.wsum[2][lane & (NW - 1)]);
    if (b == block0) carry = __builtin_amdgcn_readlane(row_incl_scan<NT>(sh.wsum[1][lane & (NW - 1)]), NW - 1);
    // the part's own range of ranks, from the waves' totals
    const int first = wave0 ? __builtin_amdgcn_readlane(x, wave0 - 1) : 0;
    const int own = __builtin_amdgcn_readlane(x, wave1 - 1) - first;
    const int own_r = low16(own), own_a = high16(own);
    const int base_r = low16(carry) + low16(first), base_a = high16(carry) + high16(first);
    const int t0 = b * kBlock<NT> + (int)threadIdx.x * 4;
    const bool emits = wave >= wave0 && wave < wave1;
    if (emits) {
      const int before = (wave ? __builtin_amdgcn_readlane(x, wave - 1) : 0) + incl - mine;
      list_tokens(t0, ret4, apx4, low16(before) - low16(first), high16(before) - high16(first), own_r, sh.list);
    }
    carry += __builtin_amdgcn_readlane(x, NW - 1);
    lds_barrier();                                           // the list is whole
    if (emits) store_tiers(target, t0, ret4, apx4);
    store_indices<NT>(target, sh.list, own_r, own_a, base_r, base_a);
    if (p.g.k) copy_rows<NT>(p.g, h, p.n_approx, sh.list, own_r, own_a, base_r, base_a);
    lds_barrier();                                           // the list may be written again
  }
}

int units_of(int seq_len) { return (seq_len + kUnit - 1) / kUnit; }

void head_parts(int seq_len, int units, HeadParams& p) {
  p.units_per_part = units;
  p.parts = (units_of(seq_len) + units - 1) / units;
}

// Kernel and workgroup size for heads of up to n tokens.  A thread's tokens are worked off one after the other, so beyond
// 4096 sixteen waves share them.  Routing of given scores, sixteen waves against eight, in us:
//     heads     2048       4096       8192        12289       16384 tokens
//       1    8.4 / 7.0  8.8 / 8.1  10.2 / 10.2  13.0 / 14.4  13.3 / 14.6
//       8    8.4 / 7.1  8.7 / 8.2  10.5 / 10.5  13.3 / 14.7  13.8 / 14.9
//      64    8.4 / 7.1  9.0 / 8.4  10.6 / 10.7  15.3 / 17.6  14.4 / 16.5
// At 8192 tokens the two are alike for any number of heads (a compression pass of 8 heads 34.2 / 34.3, of 64 106.4 / 106.2, of
// eight unequal prompts 115.6 / 115.6); a pass of 12289 tokens takes 43.4 / 46.6 with 8 heads and 160.6 / 164.9 with 64.
template <bool POOL, bool RAGGED> struct HeadKernel {
  void (*kernel)(RunArgs<HeadParams, RAGGED>);
  int threads;
  explicit HeadKernel(int n) {
    threads = n <= 4096 ? 512 : 1024;
    kernel = n <= 2048   ? route_head_kernel<512, 1, POOL, RAGGED>
             : n <= 4096 ? route_head_kernel<512, 2, POOL, RAGGED>
             : n <= 8192 ? route_head_kernel<1024, 2, POOL, RAGGED>
                         : route_head_kernel<1024, 4, POOL, RAGGED>;
  }
};

HeadParams head_params(const float* mass, const float* score_in, float* score_out, const float* eps, int n, int n_prefix, int pool_kernel,
                       int pool_mode, int n_pool, int n_approx, uint8_t* tier, int32_t* idx_retain, int32_t* idx_approx) {
  HeadParams p;
  p.src = mass ? mass : score_in; p.score = score_out; p.eps = eps;
  p.n = n; p.n_prefix = n_prefix; p.half = pool_kernel / 2; p.take_max = pool_mode == VECTOR_POOL_MAX;
  p.inv_kernel = 1.0f / (float)pool_kernel;
  p.n_pool = n_pool; p.n_approx = n_approx;
  p.tier = tier; p.idx_retain = idx_retain; p.idx_approx = idx_approx;
  p.g = GatherParams{};
  p.seq_table = nullptr; p.seq_hps = 0;
  return p;
}

}  // namespace

bool route_head_fits(int seq_len) { return seq_len <= kMaxHead; }
bool route_head_pools(int pool_kernel) { return pool_kernel / 2 <= kMaxHalf; }

int launch_route_head(int n_kv_heads, int seq_len, const float* score, const float* eps, int n_pool, int n_approx, uint8_t* tier,
                      int32_t* idx_retain, int32_t* idx_approx, const HeadPool* pool, const PackedRows* rows, hipStream_t stream) {
  if (n_pool < 1 || n_approx < 0 || n_pool < n_approx || n_pool > seq_len || !route_head_fits(seq_len) || (pool && !route_head_pools(pool->kernel))) return VECTOR_ERR_ARG;
  HeadParams p = head_params(pool ? pool->mass : nullptr, score, pool ? pool->score : nullptr, eps, seq_len, pool ? pool->n_prefix : seq_len,
                             pool ? pool->kernel : 1, pool ? pool->mode : VECTOR_POOL_AVG, n_pool, n_approx, tier, idx_retain, idx_approx);
  if (rows)
    p.g = gather_params(*rows->shape, rows->k, rows->v, idx_retain, idx_approx, n_pool - n_approx, n_approx, rows->k_ret, rows->v_ret,
                        rows->k_apx, rows->cap_retain, rows->stack);
  const int n_units = units_of(seq_len);
  head_parts(seq_len, part_units(&n_units, 1, n_kv_heads), p);
  const HeadKernel<true, false> pooling(seq_len);
  const HeadKernel<false, false> given(seq_len);
  const auto k = pool ? pooling.kernel : given.kernel;
  const RunArgs<HeadParams, false> args = {{p}};
  VEC_LAUNCH(K_ROUTE, k, dim3(p.parts, n_kv_heads), dim3(given.threads), 0, stream, args);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

size_t route_head_table_bytes(int count) { return align_up(sizeof(HeadParams) * count, 256); }

int launch_route_head_ragged(const vector_shape& s, const RaggedSeq* seqs, int count, void* tables, hipStream_t stream) {
  if (count < 1 || count > kMaxRaggedSeqs || !route_head_pools(s.pool_kernel)) return VECTOR_ERR_ARG;
  HeadParams host[kMaxRaggedSeqs];
  int n_units[kMaxRaggedSeqs], longest = 0;
  for (int b = 0; b < count; ++b) {
    n_units[b] = units_of(seqs[b].shape.seq_len);
    longest = std::max(longest, seqs[b].shape.seq_len);
  }
  const int units = part_units(n_units, count, s.n_kv_heads);
  RunArgs<HeadParams, true> args;
  std::fill(args.first, args.first + kMaxRaggedSeqs, 0xffff);
  unsigned grid = 0;
  for (int b = 0; b < count; ++b) {
    const RaggedSeq& q = seqs[b];
    const int n = q.shape.seq_len;
    if (q.n_pool < 1 || q.n_approx < 0 || q.n_pool < q.n_approx || q.n_pool > n || !route_head_fits(n)) return VECTOR_ERR_ARG;
    host[b] = head_params(score_mass(q.shape, q.score_ws), nullptr, q.score, q.eps, n, n - q.shape.window, s.pool_kernel, s.pool_mode, q.n_pool,
                          q.n_approx, q.tier, q.idx_retain, q.idx_approx);
    host[b].g = gather_params(q.shape, q.k, q.v, q.idx_retain, q.idx_approx, q.n_pool - q.n_approx, q.n_approx, q.k_ret, q.v_ret, q.k_apx,
                              q.cap_retain, nullptr);
    head_parts(n, units, host[b]);
    args.first[b] = (uint16_t)grid;
    grid += (unsigned)(host[b].parts * s.n_kv_heads);
    if (grid > 0xffff) return VECTOR_ERR_SHAPE;      // cannot be: 256 workgroups at most, or one per head, and a batch's part has fewer heads
  }
  const int rc = ragged_args(host, count, s.n_kv_heads, tables, stream, args);
  if (rc != VECTOR_OK) return rc;
  const HeadKernel<true, true> k(longest);
  VEC_LAUNCH(K_ROUTE, k.kernel, dim3(grid), dim3(k.threads), 0, stream, args);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

}  // namespace vec
