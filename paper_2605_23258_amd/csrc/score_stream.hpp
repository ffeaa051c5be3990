// The two passes over the keys (scores, and the residual riding on the second), as streams of row tiles
// through LDS.  See score_residual.hip for what they compute.
//
// Eight waves; everything that stays the same for a whole workgroup lives in the registers of the wave that
// needs it, in operand order: a 32-row block of the query rows (a "unit"; two for more than 256 rows) and
// one 32-dim block of W^T.  What streams is the token axis: tiles of 16 KB of keys (and as much of values) go
// from memory straight into a ring of LDS stages (global_load_lds, 16 bytes a lane), three tiles ahead of
// their use, with one barrier per tile.  (Where the residual's products come a tile late, rotated keys and fp32, two tiles ahead, and the
// values' blocks, outside the ring, while the tile itself is worked on: see Pass2Lds.)  The loads need no registers and no wave waits on its own trip to
// memory, so the copies run on while the matrix cores and the exponentials work.
// With keys in registers and query rows in LDS instead, a wave's next keys can only be asked for after the last product
// of the tile, and the staging (query rows, W^T two bytes at a time) takes 5 us per workgroup: the times in brackets
// below.
// Rotated keys: a tile's keys are un-rotated into LDS by all waves, and the residual's products on them are issued between the
// next tile's sines and cosines, so that a tile needs one barrier; what bounds a tile is issue (vector work 1.3 us, 48 MFMAs a
// SIMD that keep it back for 16 cycles each) and LDS (320 KB of accesses).  With a second barrier before the products, and
// the values staged with the keys, 20011 tokens x 8 heads took 2 us more, and fp32 at d = 128, which spilled 150 registers,
// 1.5 to 1.9 times as long (a pass of 2546 tokens, 8 heads, 83 us, now 44).  Tiles of half the size (more of them on their way, a
// barrier for every 32 tokens): 2.9 us per 64 tokens instead of 2.4.
// Bounds (averages of a kernel trace of back-to-back passes): 32768 tokens x 8 heads, 256 query rows: 27 us (28) for pass 1 and 38 us (39)
// for pass 2, instruction issue, at a clock of 2.0 GHz; 131072 tokens, 128 rows: 61 us (63) and 100 us (107), HBM at 4.4 and 5.4 TB/s;
// 8192 tokens: 8.4 us (9) and 12 us (19), latency.
// A lane's 16 bytes land at lane * 16, so rows cannot be padded: the 16-byte slots of a row are permuted by
// the row instead (the lane fetches the piece that belongs in its slot), which keeps 16 rows read at one
// piece in 16 different banks.
#pragma once
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace vec {

constexpr int kStreamThreads = 512, kStreamWaves = kStreamThreads / kWave;
constexpr int kStreamTileBytes = 16384;

struct PassParams {
  const void* q;        // [Hq, w, d]
  const void* k;
  const void* v;
  const void* W;
  int64_t k_sh, k_st, v_sh, v_st, w_sh;   // element strides
  int hps;              // stacked sequences: KV heads per sequence (0: one sequence); head hv of the launch is
  int64_t k_sb, v_sb;   // KV head hv % hps of sequence hv / hps, sequences k_sb / v_sb elements apart
  int n, w, R, R_pad, n_prefix;
  // Query heads of a KV head taken a group at a time (when all G * w rows do not fit at once): this
  // launch sees R rows starting at row q_row0 of the head's q_head_rows = G * w rows, and its
  // column mass is added to what the earlier groups left.
  int q_head_rows, q_row0, accumulate;
  int tokens_per_wg;     // pass 2: tokens per workgroup
  int tpc1, n_chunks;    // pass 1: tokens per chunk (one partial per row and chunk), and the number of chunks
  int chunks_per_wg;     // pass 1: chunks that one workgroup takes one after the other
  float c2;             // log2(e) / sqrt(d)
  float inv_R;
  float2* part;         // [Hkv, n_chunks, R_pad]  (reference, sum-exp against it), log2 domain
  float* mass;          // [Hkv, n]
  float* eps;           // [Hkv, n]
  float4* range;        // [Hkv, range_stride] or null: every workgroup of pass 2 leaves, over the prefix columns
                        // it stored with a positive mass m, their count and the sums of l and l * l, where
                        // l = log2(m) - log_ref; the routing's bucket launch turns them into the head's
                        // typical score range
  int range_stride;     // entries of `range` per head (the second pass's workgroups per head)
  int wgs1;             // the first pass's workgroups per head
  int64_t pos_base;     // post-RoPE keys with a position array: token t of this head is at positions[pos_base + t]
                        // (+ the sequence's share when sequences are stacked)
  // Several sequences of different lengths in one launch (template flag RAGGED, see PassArgs): a workgroup takes its
  // sequence's block.
  const PassParams* seq_table;     // the sequences' parameter blocks, where they are too many for kernel arguments
  int seq_hps;
  const float* lse;     // null, or the log-sum-exp (natural log, logits scaled by 1/sqrt(d)) of every query row,
  int64_t lse_sh;       // row r of query head hq at lse[hq * lse_sh + r]: then pass 2 needs no pass 1
  float log_ref;        // log2 of the mean mass of a prefix column, -log2(n_prefix): keeps l small
  int repeat;           // probe kernels only: times each tile's arithmetic is run on the same operands
};

// The first argument of both passes
template <bool RAGGED> using PassArgs = RunArgs<PassParams, RAGGED>;

// Which chunk of which head this workgroup takes
template <bool RAGGED>
__device__ __forceinline__ void take_chunk(PassParams& p, int& wg, int& h, bool first_pass) {
  if constexpr (RAGGED) {
    int seq;
    const int r = take_workgroup<PassArgs<true>>(p, seq);
    const int per_head = first_pass ? p.wgs1 : p.range_stride;
    h = r / per_head;
    wg = r - h * per_head;
  } else {
    xcd_chunk_head(wg, h);
  }
}

// element offset of a launch head's keys (or values), and the KV head whose W it uses
__device__ __forceinline__ int64_t head_offset(const PassParams& p, int h, int64_t seq_stride, int64_t head_stride) {
  return p.hps ? (int64_t)(h / p.hps) * seq_stride + (int64_t)(h % p.hps) * head_stride : (int64_t)h * head_stride;
}
__device__ __forceinline__ int w_head(const PassParams& p, int h) { return p.hps ? h % p.hps : h; }

template <typename T, int D> struct Stream {
  static constexpr int E = Elem<T>::kPerChunk;
  static constexpr int kRowBytes = D * (int)sizeof(T);
  static constexpr int kTileBytes = kStreamTileBytes;
  static constexpr int kTokens = kTileBytes / kRowBytes;     // tokens per tile: 64 (bf16 d = 128, fp32 d = 64), 128 or 32
  static constexpr int kSub = kTokens / 32;                  // 32-token subtiles
  static constexpr int kPieces = kRowBytes / 16;
  static constexpr int kRowsPerLoad = kWave / kPieces;       // rows that one wave-wide load brings
  static constexpr int kLoads = kTileBytes / (kWave * 16) / kStreamWaves;    // loads per wave and tile: 2
  static constexpr int NC = D / (2 * E);                     // operand chunks per row
  // Operand chunks of keys held in registers: bf16 all of a subtile's, each replaced by the next subtile's as
  // it is used up; fp32 (four slow MFMAs a chunk, twice the registers) a window of four.
  static constexpr int kWindow = sizeof(T) == 2 ? NC : 4;
  static constexpr int JB = D / 32;                          // 32-dim blocks of the value dims
  static constexpr int VP = 16 / E;                          // 16-byte pieces of a lane's 16 value dims
  // what the 16-byte slots of a row are xor-ed with
  static __device__ __forceinline__ int twist(int row) { return kPieces >= 16 ? (row & 15) : ((row >> 1) & 7); }
};

// at most `tiles` tiles of PER loads each may still be on their way
template <int PER> __device__ __forceinline__ void wait_tiles(int tiles) {
  if (tiles >= 2) wait_loads<2 * PER>();
  else if (tiles == 1) wait_loads<PER>();
  else wait_loads<0>();
}
// own LDS accesses done, then everyone's; no fence of vector memory (the tiles in flight stay in flight)
__device__ __forceinline__ void tile_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// the rows of a head (keys, or values) as a sequence of tiles, `dir` = 1 upwards or -1 downwards
template <typename T, int D> struct TileSource {
  using S = Stream<T, D>;
  const unsigned char* rows;
  const unsigned char* next;         // first row of the next tile
  int64_t st, tile_bytes;            // bytes per token and per tile (signed by the direction)
  int64_t off[S::kLoads];
  int wave, lane;
  __device__ __forceinline__ void init(const T* head, int64_t st_elems, int first_token, int dir, int wave_, int lane_) {
    rows = reinterpret_cast<const unsigned char*>(head);
    st = st_elems * (int64_t)sizeof(T);
    next = rows + (int64_t)first_token * st;
    tile_bytes = (int64_t)dir * S::kTokens * st;
    wave = wave_; lane = lane_;
#pragma unroll
    for (int i = 0; i < S::kLoads; ++i) off[i] = (int64_t)row(i) * st + piece(i) * 16;
  }
  __device__ __forceinline__ int row(int i) const { return (wave * S::kLoads + i) * S::kRowsPerLoad + lane / S::kPieces; }
  __device__ __forceinline__ int piece(int i) const { return (lane % S::kPieces) ^ S::twist(row(i)); }
  // The next tile, tokens [t0, t0 + kTokens), into the LDS tile at `lds`; rows from t_end on are copies of row t_end - 1.
  __device__ __forceinline__ void load(uint32_t lds, int t0, int t_end) {
    lds += wave * S::kLoads * 1024;
    if (__builtin_expect(t0 + S::kTokens <= t_end, 1)) {
#pragma unroll
      for (int i = 0; i < S::kLoads; ++i) load_to_lds16(lds + i * 1024, next + off[i]);
    } else {
#pragma unroll
      for (int i = 0; i < S::kLoads; ++i) load_to_lds16(lds + i * 1024, rows + (int64_t)min(t0 + row(i), t_end - 1) * st + piece(i) * 16);
    }
    next += tile_bytes;
  }
};

__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// Pure arithmetic has no position of its own in the instruction stream: the compiler
// would issue a block's MFMAs back to back and its exponentials after them.  An empty
// volatile asm that "uses" an accumulator and the running sum ties both chains to this
// point, so what is written between two pins is also issued between them.
#define VEC_PIN(acc, x) asm volatile("" : "+v"(acc), "+v"(x))
#define VEC_PIN3(acc, x, y) asm volatile("" : "+v"(acc), "+v"(x), "+v"(y))

// Which subtiles of a tile a wave works on.  NRB (4, 8 or 16) units of 32 query rows, padded with zero
// rows: with 4, waves w and w + 4 share unit w and split the subtiles; with 8, wave w takes unit w on every
// subtile; with 16, units w and w + 8.  The residual has kSub * JB products of 32 tokens x 32 dims per
// tile, one per wave, on the subtile `res_sub` that the wave works on last (where there are four, see kLastFour).
template <typename T, int D, int NRB> struct WaveWork {
  using S = Stream<T, D>;
  static constexpr int U = NRB == 16 ? 2 : 1;
  static constexpr int PH = NRB == 4 ? (S::kSub == 4 ? 2 : 1) : S::kSub;          // subtiles per wave and tile
  static constexpr int kPerSub = kStreamWaves / S::kSub;                           // waves that end on one subtile
  static constexpr int kEntries = NRB == 4 ? 4 : 8;                                // partial column sums per token
  static constexpr bool kPairs = NRB == 4;                                         // two waves share a unit
  static constexpr int kUnitSlots = kPairs ? 4 : kStreamWaves * U;                 // units that the waves hold, with those beyond the rows
  int unit, grp, first, res_sub, res_block;
  bool has_rows, has_res;
  __device__ __forceinline__ WaveWork(int wave) {
    unit = NRB == 4 ? (wave & 3) : wave;
    grp = wave >> 2;
    has_rows = !(NRB == 4 && S::kSub == 1 && grp == 1);
    first = (NRB == 4 && S::kSub > 1) ? grp * (S::kSub / 2) : 0;
    res_sub = wave / kPerSub;
    res_block = S::kSub == 1 ? (wave ^ 4) : wave % kPerSub;
    has_res = res_block < S::JB;
  }
  __device__ __forceinline__ int sub(int ph) const {
    if (ph == PH - 1) return res_sub;
    return first + ph + (first + ph >= res_sub ? 1 : 0);
  }
};

// LDS by its 32-bit address (no trip through a flat pointer's arithmetic)
__device__ __forceinline__ chunk_t lds_read16(uint32_t at) {
  const u32x4 x = *reinterpret_cast<const __attribute__((address_space(3))) u32x4*>(at);
  return make_uint4(x[0], x[1], x[2], x[3]);
}
// where this lane finds operand chunk c of its row of the first subtile, from the tile's start
template <typename T, int D> __device__ __forceinline__ uint32_t operand_at(int row, int half, int c) {
  return (uint32_t)(row * Stream<T, D>::kRowBytes + (((2 * c + half) ^ Stream<T, D>::twist(row)) * 16));
}

// the key operands of the subtile at hand
template <typename T, int D> struct KeyOperands {
  using S = Stream<T, D>;
  static constexpr bool kAll = S::kWindow == S::NC;
  chunk_t kf[S::kWindow];
  uint32_t at[kAll ? S::NC : 1];
  __device__ __forceinline__ KeyOperands(uint32_t smem0, int row, int half) {
#pragma unroll
    for (int c = 0; c < (kAll ? S::NC : 1); ++c) at[c] = smem0 + operand_at<T, D>(row, half, c);
  }
  // from here on `tile` is an offset from the first subtile of the ring's start (a multiple of the row size)
  __device__ __forceinline__ chunk_t read(uint32_t tile, int c) const { return lds_read16(kAll ? at[c] + tile : (at[0] ^ (uint32_t)(c * 32)) + tile); }
  __device__ __forceinline__ void load(uint32_t tile) {
#pragma unroll
    for (int c = 0; c < S::kWindow; ++c) kf[c] = read(tile, c);
  }
  __device__ __forceinline__ void begin(uint32_t tile) { if (!kAll) load(tile); }
  __device__ __forceinline__ const chunk_t& chunk(int c) const { return kf[c % S::kWindow]; }
  // chunk c has been used for the last time
  __device__ __forceinline__ void used(int c, uint32_t tile, uint32_t next_tile) {
    if (kAll) kf[c] = read(next_tile, c);
    else if (c + S::kWindow < S::NC) kf[c % S::kWindow] = read(tile, c + S::kWindow);
  }
};

// A wave's units of query rows, through LDS: whole rows with one load, laid out as a subtile of keys is.  (Asked for in
// operand order, 16 bytes of 64 different rows with one load, they kept a CU's address unit busy for 1.1 us per eight units.)
// Waves that share a unit (up to 128 rows) fetch half of it each, and add up half of its chunks' sums in pass 2; both are there a barrier
// later.  Both waves doing all of it kept the address unit busy for twice as long (64 of 256 loads of pass 2's first 3.4 us at 8192 tokens; a
// compression pass, us, both doing all / half each: 1024 tokens fp32 24.7 / 24.2, 8192 tokens 32.9 / 32.6, 20011 with log-sum-exp 54.3 / 53.8,
// two heads of 11469 tokens, 128 chunks each, 37.5 / 36.0).
template <typename T, int D> struct QueryUnit {
  using S = Stream<T, D>;
  static constexpr int kBytes = 32 * S::kRowBytes, kLoads = kBytes / (kWave * 16);
  // rows unit * 32 .. of the `R` at `rows`, or (PARTS 2) half of them; those beyond are copies of the last
  template <int PARTS> static __device__ __forceinline__ void load(uint32_t lds, const T* rows, int unit, int part, int R, int lane) {
#pragma unroll
    for (int j = 0; j < kLoads / PARTS; ++j) {
      const int i = PARTS == 1 ? j : part * (kLoads / PARTS) + j, row = i * S::kRowsPerLoad + lane / S::kPieces, piece = (lane % S::kPieces) ^ S::twist(row);
      load_to_lds16(lds + i * 1024, reinterpret_cast<const unsigned char*>(rows) + (size_t)min(unit * 32 + row, R - 1) * S::kRowBytes + piece * 16);
    }
  }
  // operand chunk c of the lane's row
  static __device__ __forceinline__ chunk_t read(uint32_t lds, int row, int half, int c) { return lds_read16(lds + operand_at<T, D>(row, half, c)); }
};

// ---------------------------------------------------------------------------
// pass 1: per-row softmax statistics over a chunk of tokens
// ---------------------------------------------------------------------------
constexpr int kStages1 = 4;
// LDS of pass 1: the ring, [2][4][32] float2 for the waves that share a unit, and the query rows on their way into the registers, where
// there is room for them; else in the place of the tiles after the first.  bf16 rows of 64 dims and one unit a wave: two workgroups
// fit a CU as long as they have no more than the ring; their query rows go straight into the registers.
template <typename T, int D, int NRB> struct Pass1Lds {
  static constexpr int kQueryBytes = WaveWork<T, D, NRB>::kUnitSlots * QueryUnit<T, D>::kBytes;
  static constexpr bool kThrough = !(sizeof(T) == 2 && D == 64 && NRB < 16);
  static constexpr int kRing = kStages1 * kStreamTileBytes, kShares = kRing, kSharesEnd = kRing + kStreamWaves * 32 * (int)sizeof(float2);
  static constexpr bool kApart = kSharesEnd + kQueryBytes <= (int)kMaxLdsBytes;
  static constexpr int kQuery = kApart ? kSharesEnd : kStreamTileBytes;
  static constexpr int kTotal = !kThrough ? kSharesEnd : kQuery + kQueryBytes > kSharesEnd ? kQuery + kQueryBytes : kSharesEnd;
  static_assert(kTotal <= (int)kMaxLdsBytes, "LDS");
};

template <typename T, int D, int NRB, bool RAGGED>
__global__ __launch_bounds__(kStreamThreads) void score_stats_kernel(PassArgs<RAGGED> args) {
  PassParams p = args.p;
  int wg, h;
  take_chunk<RAGGED>(p, wg, h, true);
  using S = Stream<T, D>;
  using WW = WaveWork<T, D, NRB>;
  constexpr int NC = S::NC, U = WW::U, PH = WW::PH;
  using L = Pass1Lds<T, D, NRB>;
  extern __shared__ __align__(16) unsigned char smem[];

  int chunk = wg * p.chunks_per_wg;
  const int chunk_end = min(p.n_chunks, chunk + p.chunks_per_wg);
  if (chunk >= chunk_end) return;                // as in pass 2
  const int t_begin = chunk * p.tpc1, t_end = min(p.n, chunk_end * p.tpc1);
  const int n_steps = (t_end - t_begin + S::kTokens - 1) / S::kTokens;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), half = lane >> 5, l31 = lane & 31;
  const WW ww(wave);
  float2* grp = reinterpret_cast<float2*>(smem + L::kShares);
  const uint32_t smem0 = lds_address(smem);

  TileSource<T, D> keys;
  keys.init(reinterpret_cast<const T*>(p.k) + head_offset(p, h, p.k_sb, p.k_sh), p.k_st, t_begin, 1, wave, lane);
  constexpr uint32_t kRing = kStages1 * S::kTileBytes;
  uint32_t at_fetch = 0;                         // ring position of the tile to be fetched next
  int t_fetch = t_begin, to_fetch = n_steps;     // its first token, and the tiles still to be fetched
  auto fetch = [&]() VEC_INLINE {
    keys.load(smem0 + at_fetch, t_fetch, t_end);
    at_fetch = at_fetch + S::kTileBytes == kRing ? 0 : at_fetch + S::kTileBytes;
    t_fetch += S::kTokens;
    --to_fetch;
  };
  fetch();
  // this wave's query rows: zero beyond R
  chunk_t qf[U][NC];
  int qrow[U];
  const T* q_rows = reinterpret_cast<const T*>(p.q) + ((size_t)h * p.q_head_rows + p.q_row0) * D;
  using Q = QueryUnit<T, D>;
  const uint32_t q_lds = smem0 + L::kQuery + (WW::kPairs ? ww.unit : wave * U) * Q::kBytes;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    qrow[u] = (ww.unit + 8 * u) * 32 + l31;
    if constexpr (L::kThrough) {
      Q::template load<WW::kPairs ? 2 : 1>(q_lds + u * Q::kBytes, q_rows, ww.unit + 8 * u, ww.grp, p.R, lane);
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c) qf[u][c] = load_chunk(q_rows + (size_t)min(qrow[u], p.R - 1) * D + chunk_elem_offset<T>(c, half));
    }
  }
  if constexpr (L::kThrough) {
    wait_loads<0>();
    if constexpr (WW::kPairs) tile_barrier();
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) qf[u][c] = Q::read(q_lds + u * Q::kBytes, l31, half, c);
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (qrow[u] >= p.R) qf[u][c] = make_uint4(0, 0, 0, 0);
      asm volatile("" : "+v"(qf[u][c].x), "+v"(qf[u][c].y), "+v"(qf[u][c].z), "+v"(qf[u][c].w));     // arrived: no wait on them below
    }
  if constexpr (L::kThrough && !L::kApart) tile_barrier();      // everyone's rows are out of the tiles' places
#pragma unroll
  for (int s = 1; s < kStages1 - 1; ++s)
    if (to_fetch > 0) fetch();

  // Of query row qrow[u], over this lane half's tokens: the sum of exp2(logit - m_ref).  m_ref is the
  // maximum of the row's first tile and stays: any reference does as long as the sum neither overflows nor
  // loses what it has, and a sum of 16 terms under 2^60 shows that it has not.  A block that fails that is
  // folded again against its own maximum.
  float m_ref[U], l_run[U];
  auto restart = [&]() VEC_INLINE {
#pragma unroll
    for (int u = 0; u < U; ++u) { m_ref[u] = -INFINITY; l_run[u] = 0.f; }
  };
  restart();
  auto refold = [&](const f32x16& x, int u) VEC_INLINE {
    float m0 = max3(x[0], x[1], x[2]), m1 = max3(x[8], x[9], x[10]);
    m0 = max3(m0, x[3], x[4]); m1 = max3(m1, x[11], x[12]);
    m0 = max3(m0, x[5], x[6]); m1 = max3(m1, x[13], x[14]);
    const float m_new = fmaxf(m_ref[u], fmaxf(fmaxf(m0, x[7]), fmaxf(m1, x[15])) * p.c2);     // c2 > 0: scaling commutes with max
    const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      s0 += fast_exp2(fmaf(x[v], p.c2, -m_safe));
      s1 += fast_exp2(fmaf(x[v + 1], p.c2, -m_safe));
    }
    l_run[u] = l_run[u] * fast_exp2(m_ref[u] - m_safe) + (s0 + s1);
    m_ref[u] = m_new;
  };

  auto fold_last = [&](const f32x16& x, int u) VEC_INLINE {
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      s0 += fast_exp2(fmaf(x[v], p.c2, -m_ref[u]));
      s1 += fast_exp2(fmaf(x[v + 1], p.c2, -m_ref[u]));
    }
    s0 += s1;
    if (__builtin_expect(__any(!(s0 < 1.0e18f)), 0)) refold(x, u);
    else l_run[u] += s0;
  };

  // rows = tokens, columns = query rows.  A phase runs the products of one subtile, one operand chunk at a
  // time, each followed by its share of the exponentials of the phase before: the matrix pipe works through
  // the new products while the vector ALU folds the finished ones.
  f32x16 acc[2][U];
  KeyOperands<T, D> keys_op(smem0, l31, half);
  auto phase = [&](auto cur_tag, auto fold_tag, auto refold_tag, uint32_t this_at, uint32_t next_at) VEC_INLINE {
    constexpr int kCur = decltype(cur_tag)::value;
    constexpr bool kFold = decltype(fold_tag)::value;
    if constexpr (decltype(refold_tag)::value) {     // a chunk's first products: there is no reference yet
#pragma unroll
      for (int u = 0; u < U; ++u) refold(acc[1 - kCur][u], u);
    }
    float s0[U], s1[U];
#pragma unroll
    for (int u = 0; u < U; ++u) { s0[u] = 0.f; s1[u] = 0.f; }
    keys_op.begin(this_at);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        f32x16& nx = acc[kCur][u];
        const f32x16& cu = acc[1 - kCur][u];
        if (c == 0) mma_chunk_first<T>(nx, keys_op.chunk(c), qf[u][c]);
        else mma_chunk<T>(nx, keys_op.chunk(c), qf[u][c]);
        if (u == U - 1) keys_op.used(c, this_at, next_at);
        if (kFold) {
#pragma unroll
          for (int v = c * 16 / NC; v < (c + 1) * 16 / NC; ++v) {
            const float e = fast_exp2(fmaf(cu[v], p.c2, -m_ref[u]));
            if (v & 1) s1[u] += e; else s0[u] += e;
          }
          VEC_PIN3(nx, s0[u], s1[u]);
        }
      }
    }
    if (kFold) {
      bool redo = false;
#pragma unroll
      for (int u = 0; u < U; ++u) { s0[u] += s1[u]; redo |= !(s0[u] < 1.0e18f); }
      if (__builtin_expect(__any(redo), 0)) {
#pragma unroll
        for (int u = 0; u < U; ++u) refold(acc[1 - kCur][u], u);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) l_run[u] += s0[u];
      }
    }
  };
  auto mask = [&](f32x16* x, int t0, int c_end) VEC_INLINE {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // query row (g, r) sits at position n - w + r and sees tokens <= that
      const int last = (qrow[u] < p.R) ? min(p.n_prefix + ((p.q_row0 + qrow[u]) % p.w), c_end - 1) : c_end - 1;
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (t0 + acc_row(v, half) > last) x[u][v] = -INFINITY;
    }
  };

  // byte offset of phase ph's subtile in its tile
  auto sub_at = [&](int ph) VEC_INLINE { return (uint32_t)(ww.sub(ph) * 32 * S::kRowBytes); };
  wait_tiles<S::kLoads>(min(kStages1 - 2, n_steps - 1));
  tile_barrier();
  keys_op.load(sub_at(0));
  uint32_t slot = 0;
  int t0 = t_begin, left = n_steps;            // tiles from this one on
  auto merge = [&](float& m, float& l, float m2, float l2) VEC_INLINE {
    const float mn = fmaxf(m, m2);
    const float ms = (mn == -INFINITY) ? 0.f : mn;
    l = l * fast_exp2(m - ms) + l2 * fast_exp2(m2 - ms);
    m = mn;
  };
  // four units: two waves saw a row's tokens; the first adds the other's share, left in LDS, a barrier later
  constexpr bool kPaired = NRB == 4 && S::kSub > 1;
  int finished = -1;                           // chunk whose shares are to be merged
  float m_own = 0.f, l_own = 0.f;
  auto finish_chunk = [&]() VEC_INLINE {
    if (kPaired && finished >= 0) {
      if (wave < 4) {
        const float2 o = grp[((finished & 1) * 4 + wave) * 32 + l31];
        merge(m_own, l_own, o.x, o.y);
        if (half == 0) p.part[((size_t)h * p.n_chunks + finished) * p.R_pad + qrow[0]] = make_float2(m_own, l_own);
      }
      finished = -1;
    }
  };
  // One tile.  Its successor is waited for here as well, so that the last phase can already read the next
  // phase's operands; the products of the last phase of a tile are folded during the first of the next.
  // first_tag: phases of this chunk already run (0, 1, or 2 for more).
  auto run_step = [&](auto par_tag, auto first_tag, int c_end) VEC_INLINE {
    constexpr int kPar = decltype(par_tag)::value;
    if (__builtin_expect(left > kStages1 - 2, 1)) wait_loads<(kStages1 - 3) * S::kLoads>();
    else wait_loads<0>();
    tile_barrier();                             // tile and successor are there for all, the stage before them is free
    if (to_fetch > 0) fetch();
    finish_chunk();
    const uint32_t next_slot = slot + S::kTileBytes == kRing ? 0 : slot + S::kTileBytes;
    if (ww.has_rows) {
      const bool tail = t0 + S::kTokens > min(p.n_prefix + 1, c_end);
      auto one = [&](auto ph_tag) VEC_INLINE {
        constexpr int ph = decltype(ph_tag)::value;
        if constexpr (ph < PH) {
          constexpr int cur = (kPar + ph) & 1;
          constexpr int kNth = decltype(first_tag)::value + ph;          // phases of this chunk before this one (at most two counted)
          phase(std::integral_constant<int, cur>{}, std::integral_constant<bool, (kNth > 1)>{}, std::integral_constant<bool, kNth == 1>{},
                slot + sub_at(ph), ph + 1 < PH ? slot + sub_at(ph + 1) : next_slot + sub_at(0));
          if (__builtin_expect(tail, 0)) mask(acc[cur], t0 + 32 * ww.sub(ph), c_end);
        }
      };
      one(std::integral_constant<int, 0>{});
      one(std::integral_constant<int, 1>{});
      one(std::integral_constant<int, 2>{});
      one(std::integral_constant<int, 3>{});
    }
    slot = next_slot;
    t0 += S::kTokens;
    --left;
  };
  for (; chunk < chunk_end; ++chunk) {
    const int c_end = min(p.n, (chunk + 1) * p.tpc1);
    const int steps = (c_end - chunk * p.tpc1 + S::kTokens - 1) / S::kTokens;
    restart();
    constexpr int kFlip = PH & 1;              // an odd number of phases per tile swaps the accumulators' roles
    using Zero = std::integral_constant<int, 0>;
    using One = std::integral_constant<int, 1>;
    using Many = std::integral_constant<int, 2>;
    run_step(Zero{}, Zero{}, c_end);
    if constexpr (kFlip) {                     // one phase per tile
      if (steps > 1) run_step(One{}, One{}, c_end);
      for (int i = 2; i < steps; i += 2) {
        run_step(Zero{}, Many{}, c_end);
        if (i + 1 < steps) run_step(One{}, Many{}, c_end);
      }
    } else {
      for (int i = 1; i < steps; ++i) run_step(Zero{}, Many{}, c_end);
    }
    // the last phase's products; then one (reference, sum) per row and chunk
    if (ww.has_rows) {
      const bool odd = (PH * steps - 1) & 1;   // which accumulators hold them
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (odd) fold_last(acc[1][u], u);
        else fold_last(acc[0][u], u);
      }
    }
    float2* out = p.part + ((size_t)h * p.n_chunks + chunk) * p.R_pad;     // [head][chunk][row]: rows of a chunk side by side
#pragma unroll
    for (int u = 0; u < U; ++u) merge(m_ref[u], l_run[u], __shfl_xor(m_ref[u], 32, kWave), __shfl_xor(l_run[u], 32, kWave));
    if (kPaired) {                             // the other wave's share is there after the next barrier
      if (half == 0 && wave >= 4) grp[((chunk & 1) * 4 + wave - 4) * 32 + l31] = make_float2(m_ref[0], l_run[0]);
      if (wave < 4) { m_own = m_ref[0]; l_own = l_run[0]; }
      finished = chunk;
    } else if (ww.has_rows && half == 0) {
#pragma unroll
      for (int u = 0; u < U; ++u) out[qrow[u]] = make_float2(m_ref[u], l_run[u]);
    }
  }
  if (kPaired) {
    tile_barrier();
    finish_chunk();
  }
}

// ---------------------------------------------------------------------------
// pass 2: column mass of the normalised probabilities, and/or the residual
// ---------------------------------------------------------------------------
// 16 bytes of un-rotated key elements back into operand form.  bf16 operands cannot hold
// the turned-back values exactly, so they go to the matrix core twice: the rounded value and
// the remainder of that rounding (about 2^-17 relative together).
template <typename T> struct SplitPack;
template <> struct SplitPack<bf16_t> {
  static constexpr bool kTwoParts = true;
  static __device__ __forceinline__ void run(const float* f, chunk_t& hi, chunk_t& lo) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      h[e] = pack_bf16(f[2 * e], f[2 * e + 1]);
      l[e] = pack_bf16(f[2 * e] - bf16_lo(h[e]), f[2 * e + 1] - bf16_hi(h[e]));
    }
    hi = make_uint4(h[0], h[1], h[2], h[3]);
    lo = make_uint4(l[0], l[1], l[2], l[3]);
  }
};
template <> struct SplitPack<float> {
  static constexpr bool kTwoParts = false;
  static __device__ __forceinline__ void run(const float* f, chunk_t& hi, chunk_t& lo) {
    hi = make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3]));
    lo = make_uint4(0, 0, 0, 0);
  }
};

// LDS of pass 2: a ring of stages (keys, values), the partial column sums of the last tiles, the row biases.
// Rotated keys: a ring of keys and positions; the values' blocks of the tile at hand and of the one before, each wave's own;
// the un-rotated keys of these two tiles.  Sums are added up and stored kBatch tiles at a
// time, by two waves per tile: done tile by tile, the other waves waited for that one wave's chain of LDS
// reads at every barrier (a third of the kernel's time).
template <typename T, int D, int NRB, bool MASS, bool RES, bool ROPE> struct Pass2Lds {
  using S = Stream<T, D>;
  using WW = WaveWork<T, D, NRB>;
  // bf16 rows of 64 dims fill the LDS with rotated keys and leave registers: biases are kept there, and pass through the place of
  // the second tile's un-rotated keys
  static constexpr bool kBiasRegs = WW::U == 1 || (ROPE && sizeof(T) == 2 && D == 64), kBiasInTurned = ROPE && sizeof(T) == 2 && D == 64;
  static constexpr int kPosBytes = ROPE ? S::kTokens <= 64 ? 256 : 512 : 0;
  // The residual's products a tile late, on LDS operands of their own: rotated keys, and fp32 keys (with both kinds of products
  // in one phase, on shared operands, the kernels at 128 dims spilled 99 to 176 registers: 3075 tokens x 8 heads, 64 query rows 83 us a
  // pass, now 56; 1130 tokens, two prompts, 128 rows 68 and 49; at 64 dims 3 to 11 % less now).  bf16 keys share their operands: one
  // read of LDS for both.
  static constexpr bool kLate = RES && (ROPE || sizeof(T) == 4);
  static constexpr int kStageBytes = S::kTileBytes * (RES && !kLate ? 2 : 1) + kPosBytes;
  static constexpr int kStages = ROPE ? 3 : 4;                      // kLate: the tile before stays, un-rotated (rotated keys) or as it is
  static constexpr int kFirstTiles = kLate ? 2 : kStages - 1;       // on their way before the first is worked on
  static constexpr int kValues = kStages * kStageBytes;                                  // [2][kStreamWaves] blocks of 32 rows by 32 dims
  static constexpr int kBlockBytes = 32 * 32 * (int)sizeof(T), kValuesBytes = kLate ? kStreamWaves * kBlockBytes : 0;
  static constexpr int kTurned = kValues + 2 * kValuesBytes;                             // [2]
  static constexpr int kTurnedBytes = ROPE ? S::kTileBytes * (SplitPack<T>::kTwoParts ? 2 : 1) : 0;
  static constexpr int kMassStep = MASS ? S::kSub * WW::kEntries * 32 * 4 : 0;
  static constexpr int kResStep = RES ? S::kSub * S::JB * 32 * 4 : 0;
  static constexpr int kBiasBytes = MASS ? NRB * 32 * 4 : 0;
  static constexpr int kTurns = kTurned + 2 * kTurnedBytes;                              // [D / 2] float2: rotary frequencies (hi, lo)
  static constexpr int kMassSums = kTurns + (ROPE ? D / 2 * 8 : 0);                      // [kSlots][kSub][kEntries][32]
  static constexpr int kFree = (int)kMaxLdsBytes - kMassSums - kBiasBytes;
  // a batch is stored while the two tiles after it leave their sums
  static constexpr int kBatch = kFree >= 6 * (kMassStep + kResStep) ? 4 : kFree >= 4 * (kMassStep + kResStep) ? 2 : 1;
  static constexpr int kSlots = kBatch + 2;
  static constexpr int kResSlots = kLate ? kBatch + 1 : kSlots;      // kLate: a tile's residuals come a step later, all at once
  static constexpr int kResSums = kMassSums + kSlots * kMassStep;                        // [kResSlots][kSub][JB][32]
  static constexpr int kEnd = kResSums + kResSlots * kResStep;
  static constexpr int kBias = kBiasInTurned ? kTurned + kTurnedBytes : kEnd;
  // The query rows pass through the places of the tiles after the first and of what lies behind these, until a barrier after which the
  // tiles are asked for and W and the biases are put down.  Not those of rotated fp32 keys of 128 dims: the kernels would spill
  // up to six registers more (2546 to 8192 tokens, 8 heads, 1.4 % longer).  Nor do two waves that share a unit of those rows each take
  // half of its chunks' sums: the six registers again, 35 spilled in place of 29 (8192 tokens, 8 heads, 93.7 us a compression pass
  // with halves, 88.2 without; with log-sum-exp, which has no sums to take, 71.2 and 67.1; 2546 tokens 48.9 and 47.0).
  static constexpr bool kThrough = MASS && !(ROPE && sizeof(T) == 4 && D == 128);
  static constexpr bool kHalves = kThrough && WW::kPairs;
  static constexpr int kQueryBytes = kThrough ? WW::kUnitSlots * QueryUnit<T, D>::kBytes : 0, kSharesBytes = kHalves ? 2048 : 0;
  // Where they fit the place of the column sums, which are not written before a tile's barrier, the rows go there: no barrier of
  // their own behind them, and a wave asks for its tiles as soon as its own loads are there, not when the slowest wave's are (bf16 rows of 64 dims, 8 heads,
  // a compression pass, us, in the place of tiles / here: 32768 tokens 56.4 / 55.6, five unequal prompts of up to 8000 45.4 / 44.9, 700 20.0 / 19.9; with log-sum-exp, two
  // unequal prompts of up to 7484, two query heads, 25.8 / 25.4 - and 25.4 with every wave's rows straight into its registers).
  static constexpr bool kRowsApart = kThrough && kEnd - kMassSums >= kQueryBytes + kSharesBytes;
  static constexpr int kQuery = kRowsApart ? kMassSums : kStageBytes;
  static constexpr int kW = ROPE ? kTurned : (kStages - 1) * kStageBytes;      // W on its way into the registers
  static constexpr int kUsed = kBiasInTurned ? kEnd : kEnd + kBiasBytes;
  // waves that share a unit: their shares of its rows' sums, [2][4][32] float2, behind the query rows, for as long as these
  static constexpr int kShares = kMassSums > kQuery + kQueryBytes ? kMassSums : kQuery + kQueryBytes, kSharesEnd = kShares + kSharesBytes;
  static constexpr int kTotal = kSharesEnd > kUsed ? kSharesEnd : kUsed;
  static_assert(kTotal <= (int)kMaxLdsBytes, "LDS");
  static_assert(!kRowsApart || (kQuery >= kTurns && kSharesEnd <= kEnd && (kBias >= kEnd || kBias + kBiasBytes <= kMassSums)), "of the sums' place only");
};

// x of this lane + x of the lane 32 further
__device__ __forceinline__ float add_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// PROBE: a tile's arithmetic is run p.repeat times on the operands at hand, to time the contraction code
// with memory out of the picture.  ROPE: the keys are cached after rotary position embedding; the
// residual un-rotates them (the scores use them as cached).
template <typename T, int D, int NRB, bool MASS, bool RES, bool ROPE, bool RAGGED, bool PROBE = false>
__global__ __launch_bounds__(kStreamThreads) void mass_residual_kernel(PassArgs<RAGGED> args, RopeParams rp) {
  PassParams p = args.p;
  int wg, h;
  take_chunk<RAGGED>(p, wg, h, false);
  using S = Stream<T, D>;
  using WW = WaveWork<T, D, NRB>;
  using L = Pass2Lds<T, D, NRB, MASS, RES, ROPE>;
  constexpr int NC = S::NC, U = WW::U, JB = S::JB, E = S::E, VP = S::VP;
  constexpr int PH = MASS ? WW::PH : 1;
  constexpr int kStages = L::kStages;
  extern __shared__ __align__(16) unsigned char smem[];

  const int t_begin = wg * p.tokens_per_wg, t_end = min(p.n, t_begin + p.tokens_per_wg);
  // Never taken: the grid has just the workgroups that have tokens.  But without it the kernels on rotated keys in unequal batches
  // spill 8 to 19 registers more.
  if (t_begin >= t_end) return;
  const int n_steps = (t_end - t_begin + S::kTokens - 1) / S::kTokens;
  const int mass_end = min(t_end, p.n_prefix);          // the mass of window columns is never used
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), half = lane >> 5, l31 = lane & 31;
  const WW ww(wave);
  const uint32_t smem0 = lds_address(smem);

  // Tiles go from the end of the workgroup's tokens towards their start: the first pass read them forwards
  // on the same XCD, so what is left of the keys in that L2 is the end.
  TileSource<T, D> keys, values;
  const int t_top = t_begin + (n_steps - 1) * S::kTokens;
  keys.init(reinterpret_cast<const T*>(p.k) + head_offset(p, h, p.k_sb, p.k_sh), p.k_st, t_top, -1, wave, lane);
  if (RES && !L::kLate) values.init(reinterpret_cast<const T*>(p.v) + head_offset(p, h, p.v_sb, p.v_sh), p.v_st, t_top, -1, wave, lane);
  const int32_t* positions = nullptr;
  if (ROPE && rp.positions) positions = rp.positions + p.pos_base + (p.hps ? (int64_t)(h / p.hps) * p.n : 0);
  constexpr int kPer = S::kLoads * (RES && !L::kLate ? 2 : 1) + (ROPE ? 1 : 0);
  constexpr uint32_t kRing = kStages * L::kStageBytes;
  auto token0 = [&](int step) VEC_INLINE { return t_top - step * S::kTokens; };
  uint32_t at_fetch = 0;                         // ring position of the tile to be fetched next
  int t_fetch = t_top, to_fetch = n_steps;       // its first token, and the tiles still to be fetched
  auto fetch = [&]() VEC_INLINE {
    keys.load(smem0 + at_fetch, t_fetch, t_end);
    if (RES && !L::kLate) values.load(smem0 + at_fetch + S::kTileBytes, t_fetch, t_end);
    if (ROPE) {        // positions of tokens 64 (wave % 2) .., from every wave alike; without an array any 4 bytes keep the count of loads the same
      const int half_tile = S::kTokens <= 64 ? 0 : wave & 1, t = min(t_fetch + half_tile * 64 + lane, t_end - 1);
      load_to_lds4(smem0 + at_fetch + S::kTileBytes + half_tile * 256,
                   positions ? reinterpret_cast<const void*>(positions + t) : reinterpret_cast<const void*>(p.q ? p.q : p.W));
    }
    at_fetch = at_fetch + L::kStageBytes == kRing ? 0 : at_fetch + L::kStageBytes;
    t_fetch -= S::kTokens;
    --to_fetch;
  };
  fetch();

  // ---- what stays in registers ----
  chunk_t qf[U][NC], wf[NC];
  int qrow[U];
  using Q = QueryUnit<T, D>;
  const uint32_t q_lds = smem0 + L::kQuery + (WW::kPairs ? ww.unit : wave * U) * Q::kBytes;
  if (MASS) {
    const T* q_rows = reinterpret_cast<const T*>(p.q) + ((size_t)h * p.q_head_rows + p.q_row0) * D;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      qrow[u] = (ww.unit + 8 * u) * 32 + l31;
      if constexpr (L::kThrough) {
        Q::template load<WW::kPairs ? 2 : 1>(q_lds + u * Q::kBytes, q_rows, ww.unit + 8 * u, ww.grp, p.R, lane);
      } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) qf[u][c] = load_chunk(q_rows + (size_t)min(qrow[u], p.R - 1) * D + chunk_elem_offset<T>(c, half));
      }
    }
  }
  // W^T as the M-side operand.  MFMA row m of block jb stands for value dim
  //   jb * 32 + ((m >> 2) & 1) * 16 + (m >> 3) * 4 + (m & 3),
  // which makes accumulator register v of a lane in half hf hold dim jb * 32 + hf * 16 + v: 16 dims of the
  // value row in a run.  bf16: W goes through the last stage of the ring (free until the first tile's
  // barrier) in 8 x 8 blocks turned round with v_perm; fp32: four dims of one column, a word at a time.
  constexpr bool kTurnW = RES && sizeof(T) == 2;
  unsigned char* w_lds = smem + L::kW;
  static_assert(!(ROPE && kTurnW) || D * D * 2 <= 2 * L::kTurnedBytes, "W goes through the un-rotated keys' place");
  const T* Wh = RES ? reinterpret_cast<const T*>(p.W) + (int64_t)w_head(p, h) * p.w_sh : nullptr;
  // The residual's product of this wave.  Late ones share no operands with the scores: four products a tile go to the last
  // four waves, one on each SIMD.
  constexpr bool kLate = L::kLate, kLastFour = kLate && S::kSub * JB == 4;
  const int res_sub = kLastFour ? (wave & 3) / JB : ww.res_sub, res_block = kLastFour ? (wave & 3) % JB : ww.res_block;
  const bool has_res = RES && (kLastFour ? wave >= 4 : ww.has_res);
  const int my_dim = (has_res ? res_block : 0) * 32 + ((l31 >> 2) & 1) * 16 + (l31 >> 3) * 4 + (l31 & 3);
  auto w_slot = [&](int j, int piece) VEC_INLINE { return j * S::kRowBytes + ((piece ^ ((j ^ (j >> 3)) & (S::kPieces - 1))) * 16); };
  const int wb_j0 = ((int)threadIdx.x % (D / 8)) * 8, wb_d0 = ((int)threadIdx.x / (D / 8)) * 8;
  uint4 wraw[8];
  if constexpr (kTurnW) {
    if ((int)threadIdx.x < D * D / 64) {
#pragma unroll
      for (int u = 0; u < 8; ++u) wraw[u] = load_chunk(Wh + (size_t)(wb_d0 + u) * D + wb_j0);
    }
  } else if constexpr (RES) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      uint32_t x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = reinterpret_cast<const uint32_t*>(Wh)[(size_t)((2 * c + half) * 4 + e) * D + my_dim];
      wf[c] = make_uint4(x[0], x[1], x[2], x[3]);
    }
  }
  // one bias per row: reference + log2(sum) over pass 1's chunks (a lane takes every second chunk of its
  // row; where two waves share a unit, every fourth, and a barrier later each adds the other's share), or the caller's log-sum-exp in the log2 domain of the logits; padded rows get +inf, which adds
  // exp2(-inf) = 0 to every column
  float* bias_lds = reinterpret_cast<float*>(smem + L::kBias);
  float bias_u[U];
  float2* shares = reinterpret_cast<float2*>(smem + L::kShares) + ww.unit * 32 + l31;      // [2][4][32]
  const bool shared_bias = L::kHalves && !p.lse;
  if (MASS) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float& bias = bias_u[u];
      bias = INFINITY;
      if (p.lse) {
        const int qr = p.q_row0 + min(qrow[u], p.R - 1), g = qr / p.w;
        bias = p.lse[((int64_t)h * (p.q_head_rows / p.w) + g) * p.lse_sh + (qr - g * p.w)] * kLog2e;
      } else if (L::kHalves || ww.has_rows) {
        constexpr int kBatch = L::kHalves ? 8 : 16, kApart = L::kHalves ? 4 : 2;      // 32 chunks at once
        const float2* part = p.part + (size_t)h * p.n_chunks * p.R_pad + qrow[u];
        float m = -INFINITY, l = 0.f;
        for (int c0 = L::kHalves ? half + 2 * ww.grp : half; c0 < p.n_chunks; c0 += kApart * kBatch) {
          float2 sv[kBatch];
#pragma unroll
          for (int i = 0; i < kBatch; ++i) sv[i] = part[(size_t)min(c0 + kApart * i, p.n_chunks - 1) * p.R_pad];
          float bm = m;
#pragma unroll
          for (int i = 0; i < kBatch; ++i)
            if (c0 + kApart * i < p.n_chunks) bm = fmaxf(bm, sv[i].x);
          const float bs = (bm == -INFINITY) ? 0.f : bm;
          l *= fast_exp2(m - bs);
#pragma unroll
          for (int i = 0; i < kBatch; ++i)
            if (c0 + kApart * i < p.n_chunks) l += sv[i].y * fast_exp2(sv[i].x - bs);
          m = bm;
        }
        const float m2 = __shfl_xor(m, 32, kWave), l2 = __shfl_xor(l, 32, kWave);
        const float mn = fmaxf(m, m2), ms = (mn == -INFINITY) ? 0.f : mn;
        const float sum = l * fast_exp2(m - ms) + l2 * fast_exp2(m2 - ms);
        if (L::kHalves) {
          if (half == 0) shares[ww.grp * 4 * 32] = make_float2(mn, sum);
        } else {
          bias = mn + __builtin_amdgcn_logf(sum);
        }
      }
    }
  }
  // All of it has arrived from here on: what is waited for below are tiles.  The waits count the tiles' loads back from the
  // last one issued; the counter falls in order of issue, so whatever else lies between (the stores of finish(),
  // registers spilled to scratch and read back) can make a wait longer than need be, never shorter.  Spilled
  // registers per lane (in unequal batches), with 4, 8 and 16 units: bf16 at d = 128 - - 13 (- - 42), on rotated keys - - 29 (15 8 48), at
  // d = 64 on rotated keys (- - 16); fp32 at d = 128, of 4 and 8 units, 7 10 (38 39), on rotated keys 29 22 (90 73), at d = 64 (- - 6), on
  // rotated keys (- - 13); elsewhere none.
  if (MASS) {
    if constexpr (L::kThrough) wait_loads<0>();
    if constexpr (L::kRowsApart) {
#pragma unroll
      for (int u = 0; u < U; ++u) asm volatile("" : "+v"(bias_u[u]));
      static_assert(!L::kRowsApart || kTurnW, "W's loads are waited for here as well");
#pragma unroll
      for (int u = 0; u < 8; ++u) asm volatile("" : "+v"(wraw[u].x), "+v"(wraw[u].y), "+v"(wraw[u].z), "+v"(wraw[u].w));
#pragma unroll
      for (int s = 1; s < L::kFirstTiles; ++s)
        if (to_fetch > 0) fetch();
    }
    if constexpr (L::kHalves) tile_barrier();    // everyone's shares and query rows are there
    if constexpr (L::kThrough) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < NC; ++c) qf[u][c] = Q::read(q_lds + u * Q::kBytes, l31, half, c);
    }
    if (shared_bias) {
      const float2 a = shares[0], b = shares[4 * 32];
      const float mn = fmaxf(a.x, b.x), ms = (mn == -INFINITY) ? 0.f : mn;
      bias_u[0] = mn + __builtin_amdgcn_logf(a.y * fast_exp2(a.x - ms) + b.y * fast_exp2(b.x - ms));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        if (qrow[u] >= p.R) qf[u][c] = make_uint4(0, 0, 0, 0);
        asm volatile("" : "+v"(qf[u][c].x), "+v"(qf[u][c].y), "+v"(qf[u][c].z), "+v"(qf[u][c].w));
      }
    if constexpr (L::kThrough && !L::kRowsApart) tile_barrier();      // everyone's query rows have left LDS
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (half == 0 && ww.has_rows) bias_lds[(ww.unit + 8 * u) * 32 + l31] = qrow[u] < p.R ? bias_u[u] : INFINITY;
  }
  if constexpr (L::kRowsApart) {
  } else if constexpr (kTurnW) {
#pragma unroll
    for (int u = 0; u < 8; ++u) asm volatile("" : "+v"(wraw[u].x), "+v"(wraw[u].y), "+v"(wraw[u].z), "+v"(wraw[u].w));
  } else if constexpr (RES) {
#pragma unroll
    for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(wf[c].x), "+v"(wf[c].y), "+v"(wf[c].z), "+v"(wf[c].w));
  }
  if constexpr (!L::kRowsApart) {
#pragma unroll
    for (int s = 1; s < L::kFirstTiles; ++s)
      if (to_fetch > 0) fetch();
  }
  if constexpr (kTurnW) {
    if ((int)threadIdx.x < D * D / 64) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;     // column j of two rows, the earlier one in the low half
        auto word = [&](int i) VEC_INLINE {
          const uint32_t a[4] = {wraw[2 * i].x, wraw[2 * i].y, wraw[2 * i].z, wraw[2 * i].w};
          const uint32_t b[4] = {wraw[2 * i + 1].x, wraw[2 * i + 1].y, wraw[2 * i + 1].z, wraw[2 * i + 1].w};
          return __builtin_amdgcn_perm(b[j >> 1], a[j >> 1], sel);
        };
        *reinterpret_cast<uint4*>(w_lds + w_slot(wb_j0 + j, wb_d0 / 8)) = make_uint4(word(0), word(1), word(2), word(3));
      }
    }
    tile_barrier();
#pragma unroll
    for (int c = 0; c < NC; ++c) wf[c] = *reinterpret_cast<const chunk_t*>(w_lds + w_slot(my_dim, 2 * c + half));
  }
  // a single unit's 16 biases (one per accumulator register) stay in registers; two units read them as they go (but see kBiasRegs)
  constexpr bool kBiasRegs = L::kBiasRegs;
  float bias_reg[kBiasRegs ? U : 1][16];
  auto read_bias = [&](int u, float* b) VEC_INLINE {
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(bias_lds + (ww.unit + 8 * u) * 32 + g4 * 8 + half * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) b[g4 * 4 + i] = x[i];
    }
  };
  if (MASS && kBiasRegs) {
#pragma unroll
    for (int u = 0; u < U; ++u) read_bias(u, bias_reg[kBiasRegs ? u : 0]);
  }
  // kLate: the wave's block of the values of the tile at `t0`, rows res_sub * 32 .., dims res_block * 32 ..; four (fp32: eight)
  // lanes on a row.  Nobody else reads it, so no barrier is needed between its arrival and its use.
  constexpr int kVPieces = 32 * (int)sizeof(T) / 16, kVLoads = 32 * kVPieces / kWave;
  auto values_at = [&](int step) VEC_INLINE { return (uint32_t)(L::kValues + (step & 1) * L::kValuesBytes + wave * L::kBlockBytes); };
  auto fetch_values = [&](int step, int t0) VEC_INLINE {
    const unsigned char* rows = reinterpret_cast<const unsigned char*>(reinterpret_cast<const T*>(p.v) + head_offset(p, h, p.v_sb, p.v_sh));
#pragma unroll
    for (int i = 0; i < kVLoads; ++i) {
      const int row = i * (kWave / kVPieces) + lane / kVPieces, piece = (lane % kVPieces) ^ (row / 2 % kVPieces);
      const int t = min(t0 + res_sub * 32 + row, t_end - 1);
      load_to_lds16(smem0 + values_at(step) + i * 1024, rows + ((int64_t)t * p.v_st + res_block * 32) * (int64_t)sizeof(T) + piece * 16);
    }
  };
  // ROPE: this thread un-rotates pieces tp and tp + kPieces / 2 of one token per tile
  const int turn_tok = (int)threadIdx.x / (S::kPieces / 2), tp = (int)threadIdx.x % (S::kPieces / 2);
  static_assert(S::kTokens * (S::kPieces / 2) == kStreamThreads, "a tile's pairs in one go");
  float2* turns = reinterpret_cast<float2*>(smem + L::kTurns);
  if (ROPE && (int)threadIdx.x < D / 2) turns[threadIdx.x] = make_float2(rp.turns_hi[threadIdx.x], rp.turns_lo[threadIdx.x]);

  // ---- the stream ----
  // phase p's products wait in mass_acc[p & 1] until phase p + 1 folds them; the residual's wait for the next
  // tile's first phase (in the other of two when that phase is also the one that starts the next ones)
  f32x16 mass_acc[2][U], res_acc[2];
  chunk_t vf[VP];
  if constexpr (PROBE) {
#pragma unroll
    for (int v = 0; v < 16; ++v) res_acc[0][v] = res_acc[1][v] = 0.f;
#pragma unroll
    for (int i = 0; i < VP; ++i) vf[i] = make_uint4(0, 0, 0, 0);
  }
  float st_n = 0.f, st_l = 0.f, st_ll = 0.f;   // over the columns this lane stores
  float* mass_sums = reinterpret_cast<float*>(smem + L::kMassSums);
  float* res_sums = reinterpret_cast<float*>(smem + L::kResSums);
  KeyOperands<T, D> keys_op(smem0, l31, half);
  auto sub_at = [&](int sub) VEC_INLINE { return (uint32_t)(sub * 32 * S::kRowBytes); };

  // One phase: the products of a subtile (query rows x tokens, dims x tokens), an operand
  // chunk at a time, each followed by its share of the finished products of the phase before: the
  // exponentials of mass_acc[1 - kCur] and the squared differences of the residual's against vf.
  // kAhead: operand chunks give way to the next subtile's as they are used up.
  auto phase = [&](auto cur_tag, auto new_mass_tag, auto new_res_tag, auto fold_mass_tag, auto fold_res_tag,
                   uint32_t this_at, uint32_t next_at, float& col, float& err, auto ahead_tag) VEC_INLINE {
    constexpr bool kAhead = decltype(ahead_tag)::value;
    constexpr int kCur = decltype(cur_tag)::value;
    constexpr bool kNewMass = decltype(new_mass_tag)::value, kNewRes = decltype(new_res_tag)::value;
    constexpr bool kFoldMass = decltype(fold_mass_tag)::value, kFoldRes = decltype(fold_res_tag)::value;
    float c0 = 0.f, c1 = 0.f, e0 = 0.f, e1 = 0.f;
    constexpr int kNew = PH == 1 ? kCur : 0, kOld = PH == 1 ? 1 - kCur : 0;
    if constexpr (kNewMass || kNewRes) keys_op.begin(this_at);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int lo = c * 16 / NC, hi = (c + 1) * 16 / NC;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float b[16];
        if constexpr (kFoldMass) {
          if constexpr (kBiasRegs) {
#pragma unroll
            for (int v = 0; v < 16; ++v) b[v] = bias_reg[u][v];
          } else {
            const int g4 = lo / 4;
            const f32x4 x = *reinterpret_cast<const f32x4*>(bias_lds + (ww.unit + 8 * u) * 32 + g4 * 8 + half * 4);
#pragma unroll
            for (int i = 0; i < 4; ++i) b[g4 * 4 + i] = x[i];
          }
        }
        if constexpr (kNewMass) {
          if (c == 0) mma_chunk_first<T>(mass_acc[kCur][u], qf[u][c], keys_op.chunk(c));
          else mma_chunk<T>(mass_acc[kCur][u], qf[u][c], keys_op.chunk(c));
        }
        if constexpr (kFoldMass) {
#pragma unroll
          for (int v = lo; v < hi; ++v) {
            const float e = fast_exp2(fmaf(mass_acc[1 - kCur][u][v], p.c2, -b[v]));
            if (v & 1) c1 += e; else c0 += e;
          }
          if constexpr (kNewMass) VEC_PIN3(mass_acc[kCur][u], c0, c1);
        }
      }
      if constexpr (kNewRes) {
        if (c == 0) mma_chunk_first<T>(res_acc[kNew], wf[c], keys_op.chunk(c));
        else mma_chunk<T>(res_acc[kNew], wf[c], keys_op.chunk(c));
      }
      if constexpr ((kNewMass || kNewRes) && (kAhead || !decltype(keys_op)::kAll)) keys_op.used(c, this_at, next_at);
      if constexpr (kFoldRes) {
#pragma unroll
        for (int v = lo; v < hi; ++v) {
          float f[E];
          Unpack16<T>::run(vf[v / E], f);
          const float df = f[v % E] - res_acc[kOld][v];
          if (v & 1) e1 = fmaf(df, df, e1); else e0 = fmaf(df, df, e0);
        }
        if constexpr (kNewRes) VEC_PIN3(res_acc[kNew], e0, e1);
        else if constexpr (kNewMass) VEC_PIN3(mass_acc[kCur][0], e0, e1);
      }
    }
    col = c0 + c1;
    err = e0 + e1;
  };
  const int entry = NRB == 4 ? ww.unit : wave;
  // sums_slot: the slot of the tile at hand, last_slot: of the tile before it
  int sums_slot = 0, last_slot = 0;
  auto leave_mass = [&](int slot, int sub, float col) VEC_INLINE {
    col = add_halves(col);
    if (half == 0) mass_sums[((slot * S::kSub + sub) * WW::kEntries + entry) * 32 + l31] = col;
  };
  auto leave_res = [&](int slot, float err) VEC_INLINE {
    err = add_halves(err);
    if (half == 0) res_sums[((slot * S::kSub + res_sub) * JB + res_block) * 32 + l31] = err;
  };
  auto res_slot = [&](int step, int slot) VEC_INLINE { return kLate ? (int)((uint32_t)step % (uint32_t)L::kResSlots) : slot; };
  // the finished sums of `count` tiles from tile `step` (slot `slot`) on, each added in one fixed order and stored
  auto finish = [&](int step, int slot, int count) VEC_INLINE {
    const int mine = wave % L::kBatch;
    if (wave >= 2 * L::kBatch || mine >= count) return;
    step += mine;
    slot += mine;
    if (slot >= L::kSlots) slot -= L::kSlots;
    const bool both = L::kBatch * 2 > kStreamWaves || !(MASS && RES);
    const bool do_mass = MASS && (both || wave < L::kBatch), do_res = RES && (both || wave >= L::kBatch);
    if (both && wave >= L::kBatch) return;
#pragma unroll
    for (int i = 0; i < (S::kTokens + 63) / 64; ++i) {
      const int tok = i * 64 + lane, t = token0(step) + tok;
      if (S::kTokens < 64 && tok >= S::kTokens) return;
      const int at = slot * S::kSub + (tok >> 5), res_at = res_slot(step, slot) * S::kSub + (tok >> 5);
      if (do_mass) {
        float m = 0.f;
#pragma unroll
        for (int x = 0; x < WW::kEntries; ++x) m += mass_sums[(at * WW::kEntries + x) * 32 + (tok & 31)];
        m *= p.inv_R;
        if (t < mass_end) {
          float* dst = p.mass + (size_t)h * p.n + t;
          if (p.accumulate) m += *dst;
          *dst = m;
          if (m > 0.f) {
            const float l = __log2f(m) - p.log_ref;
            st_n += 1.f;
            st_l += l;
            st_ll = fmaf(l, l, st_ll);
          }
        }
      }
      if (do_res) {
        float e = 0.f;
#pragma unroll
        for (int x = 0; x < JB; ++x) e += res_sums[(res_at * JB + x) * 32 + (tok & 31)];
        if (t < t_end) p.eps[(size_t)h * p.n + t] = e;
      }
    }
  };
  auto read_values = [&](uint32_t tile) VEC_INLINE {
    if constexpr (kLate) {
#pragma unroll
      for (int i = 0; i < VP; ++i) vf[i] = lds_read16(smem0 + tile + (uint32_t)((l31 * kVPieces + ((half * VP + i) ^ (l31 / 2 % kVPieces))) * 16));
      return;
    }
    const int row = res_sub * 32 + l31;
#pragma unroll
    for (int i = 0; i < VP; ++i) {
      const int piece = res_block * (32 / E) + half * VP + i;
      vf[i] = lds_read16(smem0 + tile + (uint32_t)(row * S::kRowBytes + ((piece ^ S::twist(row)) * 16)));
    }
  };
  // kLate: the residual's products of tile `step`, operand chunk by operand chunk, each read kOpsAhead chunks before its use (read
  // when it is used, every product waited for its trip to LDS: 2.6 us a tile, now 2.4); and the finished ones against the
  // tile's values
  auto turned_at = [&](int step) VEC_INLINE { return (uint32_t)(L::kTurned + (step & 1) * L::kTurnedBytes); };
  constexpr int kOpsAhead = 2;
  struct Products { chunk_t hi[NC], lo[NC]; };
  uint32_t tile = 0, tile_before = 0;            // the tile at hand in the ring, and the one before it
  auto read_turned = [&](Products& o, int step, int c) VEC_INLINE {
    const uint32_t at = (ROPE ? turned_at(step) : tile_before) + sub_at(res_sub);
    o.hi[c] = keys_op.read(at, c);
    if (ROPE && SplitPack<T>::kTwoParts) o.lo[c] = keys_op.read(at + (uint32_t)S::kTileBytes, c);
  };
  auto product = [&](Products& o, int step, int c) VEC_INLINE {
    if (c + kOpsAhead < NC) read_turned(o, step, c + kOpsAhead);
    if (c == 0) mma_chunk_first<T>(res_acc[0], wf[c], o.hi[c]);
    else mma_chunk<T>(res_acc[0], wf[c], o.hi[c]);
    if (ROPE && SplitPack<T>::kTwoParts) mma_chunk<T>(res_acc[0], wf[c], o.lo[c]);
  };
  auto products = [&](int step) VEC_INLINE {
    Products ops;
#pragma unroll
    for (int c = 0; c < kOpsAhead; ++c) read_turned(ops, step, c);
#pragma unroll
    for (int c = 0; c < NC; ++c) product(ops, step, c);
  };
  auto squares = [&]() VEC_INLINE {
    float e0 = 0.f, e1 = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      float f[E];
      Unpack16<T>::run(vf[v / E], f);
      const float df = f[v % E] - res_acc[0][v];
      if (v & 1) e1 = fmaf(df, df, e1); else e0 = fmaf(df, df, e0);
    }
    return e0 + e1;
  };
  // The un-rotated keys of the tile (rounded values, then the remainders), in the layout of a tile, into one of two places;
  // with products: meanwhile the residual's of the tile before, out of the other.
  auto unrotate = [&](int step, uint32_t tile, auto products_tag) VEC_INLINE {
    constexpr bool kProducts = decltype(products_tag)::value;
    const int tok = turn_tok, x = S::twist(tok);
    const int at_a = tok * S::kRowBytes + ((tp ^ x) * 16), at_b = tok * S::kRowBytes + (((tp + S::kPieces / 2) ^ x) * 16);
    const chunk_t ra = lds_read16(smem0 + tile + at_a), rb = lds_read16(smem0 + tile + at_b);
    Products ops;
    if constexpr (kProducts) {
#pragma unroll
      for (int c = 0; c < kOpsAhead; ++c) read_turned(ops, step - 1, c);
    }
    const int t = min(token0(step) + tok, t_end - 1);
    const int at_pos = reinterpret_cast<const int*>(smem + tile + S::kTileBytes)[tok];
    // pairs (x[i], x[i + D/2]): E frequencies in a row; pairs (x[2i], x[2i+1]): half of them, and as many D / 4 further
    f32x4 fr[E / 2];
#pragma unroll
    for (int i = 0; i < E / 2; ++i)
      fr[i] = reinterpret_cast<const f32x4*>(turns)[rp.interleaved ? tp * (E / 4) + (i < E / 4 ? i : i - E / 4 + D / 8) : tp * (E / 2) + i];
    const float pos = (float)((positions ? at_pos : t) + rp.pos_offset);
    float a[E], b[E];
    Unpack16<T>::run(ra, a);
    Unpack16<T>::run(rb, b);
    // the pairs as (a[e], b[e]); moved about, and back, where they lie side by side
    if (rp.interleaved) {                        // uniform
      asm volatile("; pairs side by side");      // a branch: as selects the moves cost everyone
      float c[2 * E];
#pragma unroll
      for (int e = 0; e < E; ++e) { c[e] = a[e]; c[E + e] = b[e]; }
#pragma unroll
      for (int e = 0; e < E; ++e) { a[e] = c[2 * e]; b[e] = c[2 * e + 1]; }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      if constexpr (kProducts) {
#pragma unroll
        for (int c = e * NC / E; c < (e + 1) * NC / E; ++c) product(ops, step - 1, c);
      }
      float cs, sn;
      rotary_cos_sin(pos, fr[e / 2][2 * (e % 2)], fr[e / 2][2 * (e % 2) + 1], cs, sn);
      rotary_back(a[e], b[e], cs, sn, a[e], b[e]);
      if constexpr (kProducts) VEC_PIN3(res_acc[0], a[e], b[e]);
    }
    if (rp.interleaved) {
      asm volatile("; and back");
      float c[2 * E];
#pragma unroll
      for (int e = 0; e < E; ++e) { c[2 * e] = a[e]; c[2 * e + 1] = b[e]; }
#pragma unroll
      for (int e = 0; e < E; ++e) { a[e] = c[e]; b[e] = c[E + e]; }
    }
    chunk_t ha, la, hb, lb;
    SplitPack<T>::run(a, ha, la);
    SplitPack<T>::run(b, hb, lb);
    unsigned char* hi = smem + turned_at(step);
    *reinterpret_cast<chunk_t*>(hi + at_a) = ha;
    *reinterpret_cast<chunk_t*>(hi + at_b) = hb;
    if (SplitPack<T>::kTwoParts) {
      *reinterpret_cast<chunk_t*>(hi + S::kTileBytes + at_a) = la;
      *reinterpret_cast<chunk_t*>(hi + S::kTileBytes + at_b) = lb;
    }
  };
  using No = std::false_type;
  using Yes = std::true_type;
  const bool has_mass = MASS && ww.has_rows;
  const int sub0 = ww.sub(MASS ? 0 : WW::PH - 1);
  wait_tiles<kPer>(min(L::kFirstTiles - 1, n_steps - 1));
  if constexpr (!kLate) {
    tile_barrier();
    keys_op.load(sub_at(sub0));
  }
  int step = 0, batch0 = 0, batch0_slot = 0;    // first tile whose sums are not stored yet, and its slot
  // One tile.  Its successor is waited for here as well, so that the last phase can already read the next
  // phase's operands; the products of the last phase of a tile are folded during the first of the next.
  auto run_step = [&](auto par_tag, auto first_tag) VEC_INLINE {
    constexpr int kPar = decltype(par_tag)::value;
    constexpr bool kFirst = decltype(first_tag)::value;
    bool fetched = true;
    if constexpr (kLate) {
      tile_barrier();                           // the tile is there for all, and the un-rotated one before it; a stage is free
      if (decltype(keys_op)::kAll && has_mass) keys_op.load(tile + sub_at(sub0));
      fetched = to_fetch > 0;
      if (fetched) fetch();
      if (has_res) fetch_values(step, token0(step));
    } else {
      if (__builtin_expect(n_steps - step > kStages - 2, 1)) wait_loads<(kStages - 3) * kPer>();
      else wait_loads<0>();
      tile_barrier();                           // tile and successor are there for all, the stage before them is free
      if (to_fetch > 0) fetch();
    }
    if (__builtin_expect(step == batch0 + L::kBatch + 1, 0)) {
      finish(batch0, batch0_slot, L::kBatch);
      batch0 += L::kBatch;
      batch0_slot += L::kBatch;
      if (batch0_slot >= L::kSlots) batch0_slot -= L::kSlots;
    }
    const uint32_t next_tile = tile + L::kStageBytes == kRing ? 0 : tile + L::kStageBytes;
    if constexpr (ROPE) {
      if (!kFirst && has_res) unrotate(step, tile, std::integral_constant<bool, !kFirst>{});
      else unrotate(step, tile, No{});
    } else if constexpr (kLate && !kFirst) {
      if (has_res) products(step - 1);
    }
    for (int rep = 0; rep < (PROBE ? p.repeat : 1); ++rep) {
      // the products of the residual start in the last phase, together with the last subtile's scores; those of rotated keys
      // in the next tile's step, beside its un-rotation
      constexpr bool kResWithMass = RES && !kLate;
      auto one = [&](auto ph_tag) VEC_INLINE {
        constexpr int ph = decltype(ph_tag)::value;
        if constexpr (ph < PH) {
          constexpr int cur = (kPar + ph) & 1;
          constexpr bool kLast = ph == PH - 1;
          constexpr bool kFold = PROBE || !(kFirst && ph == 0);
          const uint32_t here = tile + sub_at(ww.sub(MASS ? ph : WW::PH - 1));
          const uint32_t next = kLast ? (PROBE && rep + 1 < p.repeat ? tile : next_tile) + sub_at(sub0) : tile + sub_at(ww.sub(MASS ? ph + 1 : 0));
          float col, err;
          using Cur = std::integral_constant<int, cur>;
          using FoldM = std::integral_constant<bool, MASS && kFold>;
          using FoldR = std::integral_constant<bool, RES && !kLate && kFold && ph == 0>;
          using Ahead = std::integral_constant<bool, !(kLate && kLast)>;
          using NewR = std::integral_constant<bool, kResWithMass && kLast>;
          constexpr bool kAll = !kLate && (!RES || S::kSub * JB >= kStreamWaves) && !(NRB == 4 && S::kSub == 1);      // every wave has products of both kinds
          static_assert(kLate || kAll || !RES, "products of one kind alone are for late residuals");
          if constexpr (kLate) {
            if (has_mass) phase(Cur{}, std::integral_constant<bool, MASS>{}, No{}, FoldM{}, No{}, here, next, col, err, Ahead{});
          } else {
            if (kAll || has_mass) phase(Cur{}, std::integral_constant<bool, MASS>{}, NewR{}, FoldM{}, FoldR{}, here, next, col, err, Yes{});
          }
          if constexpr (FoldM::value) {
            if (kAll || has_mass) leave_mass(ph == 0 ? last_slot : sums_slot, ww.sub(ph == 0 ? PH - 1 : ph - 1), col);
          }
          if constexpr (FoldR::value) {
            if constexpr (PROBE) asm volatile("" : "+v"(err));
            if ((kAll || has_res) && (!PROBE || (rep == 0 && step > 0))) leave_res(last_slot, err);
          }
        }
      };
      one(std::integral_constant<int, 0>{});
      one(std::integral_constant<int, 1>{});
      one(std::integral_constant<int, 2>{});
      one(std::integral_constant<int, 3>{});
      if constexpr (kLate) {
        // the next tile, and the values of the one before, were asked for a step ago, before what this step asked for
        if (has_res) {
          if (fetched) wait_loads<kPer + kVLoads>(); else wait_loads<kVLoads>();
        } else {
          if (fetched) wait_loads<kPer>(); else wait_loads<0>();
        }
        if (!kFirst && has_res) {
          read_values(values_at(step - 1));
          leave_res(res_slot(step - 1, last_slot), squares());
        }
      }
      if (!kLate && has_res) read_values(tile + S::kTileBytes);
    }
    tile_before = tile;
    tile = next_tile;
    last_slot = sums_slot;
    if (++sums_slot == L::kSlots) sums_slot = 0;
    ++step;
  };
  constexpr int kFlip = PH & 1;
  run_step(std::integral_constant<int, 0>{}, Yes{});
  if constexpr (kFlip) {
    for (int i = 1; i < n_steps; i += 2) {
      run_step(std::integral_constant<int, 1>{}, No{});
      if (i + 1 < n_steps) run_step(std::integral_constant<int, 0>{}, No{});
    }
  } else {
    for (int i = 1; i < n_steps; ++i) run_step(std::integral_constant<int, 0>{}, No{});
  }
  {                                            // the last phase's products
    float col = 0.f, err = 0.f;
    if (has_mass) {
      const bool odd = (PH * n_steps - 1) & 1;
      if (odd) phase(std::integral_constant<int, 0>{}, No{}, No{}, Yes{}, No{}, 0u, 0u, col, err, Yes{});
      else phase(std::integral_constant<int, 1>{}, No{}, No{}, Yes{}, No{}, 0u, 0u, col, err, Yes{});
      leave_mass(last_slot, ww.sub(PH - 1), col);
    }
    if constexpr (kLate) {
      wait_loads<0>();
      tile_barrier();                            // the last tile's un-rotated keys are there
      if (has_res) {
        products(n_steps - 1);
        read_values(values_at(n_steps - 1));
        leave_res(res_slot(n_steps - 1, last_slot), squares());
      }
    } else if (has_res) {
      if ((n_steps - 1) & 1) phase(std::integral_constant<int, 0>{}, No{}, No{}, No{}, Yes{}, 0u, 0u, col, err, Yes{});
      else phase(std::integral_constant<int, 1>{}, No{}, No{}, No{}, Yes{}, 0u, 0u, col, err, Yes{});
      leave_res(last_slot, err);
    }
  }
  tile_barrier();
  while (batch0 < n_steps) {                    // at most two rounds
    finish(batch0, batch0_slot, min(L::kBatch, n_steps - batch0));
    batch0 += L::kBatch;
    batch0_slot += L::kBatch;
    if (batch0_slot >= L::kSlots) batch0_slot -= L::kSlots;
  }
  if (MASS && p.range) {                      // uniform: the workgroup's sums, waves added in one fixed order
    st_n = wave_sum_dpp(st_n);
    st_l = wave_sum_dpp(st_l);
    st_ll = wave_sum_dpp(st_ll);
    float* part = bias_lds;                    // every wave has read its biases for the last time
    tile_barrier();
    if (lane == 0) { part[3 * wave] = st_n; part[3 * wave + 1] = st_l; part[3 * wave + 2] = st_ll; }
    tile_barrier();
    if (threadIdx.x == 0) {
      float a = 0.f, b = 0.f, c = 0.f;
#pragma unroll
      for (int w = 0; w < kStreamWaves; ++w) { a += part[3 * w]; b += part[3 * w + 1]; c += part[3 * w + 2]; }
      p.range[(size_t)h * p.range_stride + wg] = make_float4(a, b, c, 0.f);
    }
  }
}

// ---------------------------------------------------------------------------
// launching: the kernels for one element type and head size
// ---------------------------------------------------------------------------
// The parameters of one pair of passes; what decides the kernels is the same for every sequence of a ragged launch.
struct PassLaunch {
  PassParams pp;
  int units;                 // 32-row units of query rows the kernels are built for: 4, 8 or 16
  dim3 grid1, grid2;
  uint16_t first1[kMaxRaggedSeqs], first2[kMaxRaggedSeqs];      // PassArgs::first of the two launches
  bool do_mass, do_res, use_rope;
  RopeParams rp;
};

template <typename T, int D, int NRB, bool RAGGED>
int launch_passes_units(PassArgs<RAGGED>& a, const PassLaunch& L, hipStream_t stream) {
  using Args = PassArgs<RAGGED>;
  const dim3 grid1 = L.grid1, grid2 = L.grid2;
  if (L.do_mass && !L.pp.lse) {               // pass 1; not needed when the caller brings the rows' log-sum-exp
    constexpr size_t lds = Pass1Lds<T, D, NRB>::kTotal;
    auto k1 = score_stats_kernel<T, D, NRB, RAGGED>;
    VEC_HIP(set_max_lds(reinterpret_cast<const void*>(k1), lds));
    if constexpr (RAGGED) std::copy(L.first1, L.first1 + kMaxRaggedSeqs, a.first);
    VEC_LAUNCH(K_SCORE_STATS, k1, grid1, dim3(kStreamThreads), lds, stream, a);
  }
  void (*k2)(Args, RopeParams);
  size_t lds;
  if (L.do_mass && L.do_res) {
    k2 = L.use_rope ? mass_residual_kernel<T, D, NRB, true, true, true, RAGGED> : mass_residual_kernel<T, D, NRB, true, true, false, RAGGED>;
    lds = L.use_rope ? Pass2Lds<T, D, NRB, true, true, true>::kTotal : Pass2Lds<T, D, NRB, true, true, false>::kTotal;
  } else if constexpr (RAGGED) {
    return VECTOR_ERR_ARG;
  } else if (L.do_mass) {
    k2 = mass_residual_kernel<T, D, NRB, true, false, false, false>;
    lds = Pass2Lds<T, D, NRB, true, false, false>::kTotal;
  } else {
    k2 = L.use_rope ? mass_residual_kernel<T, D, 4, false, true, true, false> : mass_residual_kernel<T, D, 4, false, true, false, false>;
    lds = L.use_rope ? Pass2Lds<T, D, 4, false, true, true>::kTotal : Pass2Lds<T, D, 4, false, true, false>::kTotal;
  }
  VEC_HIP(set_max_lds(reinterpret_cast<const void*>(k2), lds));
  if constexpr (RAGGED) std::copy(L.first2, L.first2 + kMaxRaggedSeqs, a.first);
  VEC_LAUNCH(K_MASS_RESIDUAL, k2, grid2, dim3(kStreamThreads), lds, stream, a, L.rp);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

// units of query rows that fit the registers of a workgroup (two per wave; fp32 operands of 128 dims: one)
template <typename T, int D> constexpr int kMaxUnits = (sizeof(T) == 4 && D == 128) ? 8 : 16;

template <typename T, int D, bool RAGGED>
int launch_passes(PassArgs<RAGGED>& a, const PassLaunch& L, hipStream_t stream) {
  if (L.units == 4 || !L.do_mass) return launch_passes_units<T, D, 4, RAGGED>(a, L, stream);
  if (L.units == 8) return launch_passes_units<T, D, 8, RAGGED>(a, L, stream);
  if constexpr (kMaxUnits<T, D> == 16) {
    if (L.units == 16) return launch_passes_units<T, D, 16, RAGGED>(a, L, stream);
  }
  return VECTOR_ERR_SHAPE;
}

template <typename T, int D>
int launch_probe(const PassLaunch& L, hipStream_t stream) {
  auto k2 = mass_residual_kernel<T, D, 4, false, true, false, false, true>;
  constexpr size_t lds = Pass2Lds<T, D, 4, false, true, false>::kTotal;
  VEC_HIP(set_max_lds(reinterpret_cast<const void*>(k2), lds));
  VEC_LAUNCH(K_MASS_RESIDUAL, k2, L.grid2, dim3(kStreamThreads), lds, stream, (PassArgs<false>{{L.pp}}), L.rp);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

#ifndef VEC_DEFINE_PASSES
extern template int launch_passes<bf16_t, 128, false>(PassArgs<false>&, const PassLaunch&, hipStream_t);
extern template int launch_passes<bf16_t, 128, true>(PassArgs<true>&, const PassLaunch&, hipStream_t);
extern template int launch_passes<bf16_t, 64, false>(PassArgs<false>&, const PassLaunch&, hipStream_t);
extern template int launch_passes<bf16_t, 64, true>(PassArgs<true>&, const PassLaunch&, hipStream_t);
extern template int launch_passes<float, 128, false>(PassArgs<false>&, const PassLaunch&, hipStream_t);
extern template int launch_passes<float, 128, true>(PassArgs<true>&, const PassLaunch&, hipStream_t);
extern template int launch_passes<float, 64, false>(PassArgs<false>&, const PassLaunch&, hipStream_t);
extern template int launch_passes<float, 64, true>(PassArgs<true>&, const PassLaunch&, hipStream_t);
extern template int launch_probe<bf16_t, 128>(const PassLaunch&, hipStream_t);
extern template int launch_probe<bf16_t, 64>(const PassLaunch&, hipStream_t);
#endif

}  // namespace vec
