// Least-squares value map (Section 3.1): W_h = argmin_W || K_h W - V_h ||_F^2, no intercept,
// from m calibration tokens per KV head, through the normal equations
//   (K^T K) W = K^T V.
//
//   gram_kernel / gram_f32_kernel : grid (token chunks, kv heads).  The two d x d products on the matrix
//                  cores, fp32 accumulation inside a chunk; one fp32 partial pair per chunk.
//   gram_reduce_kernel : the chunks' partials summed in fp64: four quarters in chunk order, then their sum.
//   solve_kernel : grid (d / 16 column blocks, heads).  Blocked fp64 Cholesky of K^T K with the column
//                  block of K^T V riding along, then the backward substitution; all on fp64 matrix
//                  instructions out of LDS.
// At 65536 tokens x 8 heads, d = 128 (268 MB of keys and values): 58 + 7 + 23 us (products, sums, solve; averages over inputs in turn).
#include <algorithm>

#include "common.hpp"
#include "launch.hpp"

namespace vec {

namespace {

constexpr int kCalThreads = 256;
constexpr int kCalTile = 128;                // chunks are multiples of the longest tile; 256 for bf16 keys of 64 dims
constexpr int kCalMaxChunks = 64;
constexpr int kCalMinTokens = 256;
constexpr int kCalMaxTokens = 2048;           // bf16
constexpr int kCalCus = 256;

typedef __attribute__((ext_vector_type(4))) double f64x4;

struct CalParams {
  const void* k; const void* v;
  int64_t k_sh, k_st, v_sh, v_st;           // element strides
  int m;                                    // calibration tokens per head
  int tokens_per_chunk, n_chunks;
  float* part;                              // [Hkv, n_chunks, 2, d, d] fp32: K^T K, then K^T V
  double* sums;                             // [Hkv, tiles, 16, 16] fp64: what solve_kernel loads, in its tile order
  void* W;                                  // [Hkv, d, d] out
};

// ---------------------------------------------------------------------------
// bf16 inputs.  Both products contract over tokens, so an MFMA operand is a run of eight tokens of
// one dim: the tiles are turned round on their way into LDS.  A thread takes an 8 x 8 block (eight
// 16-byte loads, one per token), swaps it with one v_perm per output word and stores eight 16-byte
// runs; every operand is then one 16-byte LDS read (reading a [token][dim] tile down its columns took
// eight 2-byte reads per operand, and those reads bound the launch).  A row of LDS holds one dim's tokens
// of the tile; the 16-byte slots of a row are permuted by the dim so that neither the stores (dims
// eight apart) nor the operand reads (dims next to each other) meet in a bank.
// One workgroup of eight waves per CU: four take K^T K, four K^T V, a 32-row block each (d = 128; for d = 64 two and two,
// and the other four the second half of the tile's tokens).  The tile after next is requested as soon as the next one's
// registers are in LDS, so that the memory is never waited for by a whole CU.
// An accumulator sums 128 tokens and is then added to a total: the errors of longer runs on the matrix cores need not average
// out over chunks (the diagonal of K^T K of normal keys comes out 6e-8 too large in every chunk of 1024 tokens, 6e-9 in runs of
// 128), those of the additions to the total do.  A total takes at most 16 of them (kCalMaxTokens; beyond 64 chunks a head m / 8192).
// Relative error of that diagonal against 64 bits (root mean square): one run over 1024 tokens (256 for few heads and tokens) / runs
// of 512 in chunks as long as one workgroup per CU makes them / this:
//   8 heads x 12000 tokens 1.2e-8 / 3.4e-8 / 1.0e-8, x 65536 6.4e-8 / 4.3e-8 / 1.2e-8; 32 x 65536 6.4e-8 / 4.7e-8 / 1.2e-8;
//   96 x 65536 6.6e-8 / 8.3e-8 / 1.2e-8; 256 x 4096 9.9e-8 / 7.5e-8 / 4.5e-8, x 32768 7.0e-8 / 11.4e-8 / 1.6e-8.
// All elements, keys and values of one sign, in units of the factors' norms: 8 x 12000 8e-9 / 11e-9 / 6e-9, x 65536 23e-9 / 12e-9 / 11e-9.
// d = 64: the two halves' totals and last accumulators are added in 64 bits and rounded once: 8 x 12000 (K^T K, K^T V) 6.6e-9 and 6.9e-9;
// rounded three times 8.1e-9 and 8.6e-9, chunks of 256 tokens in one run 8.9e-9 and 7.0e-9.
// Bound: HBM, every key and value once and 27 MB of partials: 58 us at 65536 tokens x 8 heads, inputs in turn (5.1 TB/s; 53.4 at
// best, 5.5; a plain copy moves 5.3).  Two workgroups of four waves on a CU, each with both products and chunks of 1024 tokens: 64 us (58 at best), and 12 in
// place of 7 for the sums of twice the partials; 1474 tokens x 4 heads, d = 64: 22.4 us for the fit, 17.9 with these.
// ---------------------------------------------------------------------------
constexpr int kGramThreads = 512;
template <int D> struct GramTile {
  static constexpr int kTokens = 128 * 128 / D;                   // one 8 x 8 block per thread and tile
  static constexpr int kOctets = kTokens / 8;
  static constexpr int kRowBytes = kTokens * 2;
  static constexpr int kBytes = D * kRowBytes;
  static __device__ __forceinline__ int at(int dim, int octet) {
    return dim * kRowBytes + ((octet ^ (((dim >> 3) * (128 / D) ^ dim) & 15)) * 16);
  }
};

template <int D>
__global__ __launch_bounds__(kGramThreads) void gram_kernel(CalParams p) {
  using T = bf16_t;
  using TL = GramTile<D>;
  constexpr int JB = D / 32;
  constexpr int kBlocks = kGramThreads / 2;                       // 8 x 8 blocks of K, and of V, per tile
  static_assert((D / 8) * TL::kOctets == kBlocks, "one block per thread");
  constexpr int kShares = kGramThreads / kWave / (2 * JB);        // waves that share a block row of a product, by tokens
  constexpr int kSteps = TL::kTokens / 16 / kShares;              // 16-token steps of a tile per wave
  extern __shared__ __align__(16) unsigned char gram_lds[];       // [buffer][K, V][kBytes]

  const int h = blockIdx.y, chunk = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l31 = lane & 31, half = lane >> 5;
  const int ib = wave % JB, share = wave / (2 * JB);
  const bool is_c = (wave / JB) & 1;
  // this thread's block of a tile: K or V, eight dims, eight tokens
  const bool is_v = (int)threadIdx.x >= kBlocks;
  const int bi = (int)threadIdx.x % kBlocks, dims0 = (bi % (D / 8)) * 8, octet = bi / (D / 8);
  const T* src = (is_v ? reinterpret_cast<const T*>(p.v) + (int64_t)h * p.v_sh : reinterpret_cast<const T*>(p.k) + (int64_t)h * p.k_sh) + dims0;
  const int64_t st = is_v ? p.v_st : p.k_st;
  const int c_begin = chunk * p.tokens_per_chunk;
  const int c_end = min(p.m, c_begin + p.tokens_per_chunk);
  const int n_tiles = (c_end - c_begin + TL::kTokens - 1) / TL::kTokens;

  f32x16 acc[JB], total[JB];
#pragma unroll
  for (int jb = 0; jb < JB; ++jb)
#pragma unroll
    for (int x = 0; x < 16; ++x) total[jb][x] = 0.f;

  uint4 raw[8];
  auto fetch = [&](int tile) {
    const int t0 = c_begin + tile * TL::kTokens + octet * 8;
#pragma unroll
    for (int u = 0; u < 8; ++u) raw[u] = load_chunk(src + (int64_t)min(t0 + u, p.m - 1) * st);
  };
  // rows past the chunk are staged as zeros: they add nothing to either product
  auto stash = [&](int tile, int buf) {
    const int t0 = c_begin + tile * TL::kTokens + octet * 8;
    if (t0 + 8 > c_end) {
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (t0 + u >= c_end) raw[u] = make_uint4(0, 0, 0, 0);
    }
    unsigned char* to = gram_lds + (buf * 2 + (is_v ? 1 : 0)) * TL::kBytes;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;   // dim j of two tokens, the earlier one in the low half
      auto word = [&](int i) {
        const uint32_t a[4] = {raw[2 * i].x, raw[2 * i].y, raw[2 * i].z, raw[2 * i].w};
        const uint32_t b[4] = {raw[2 * i + 1].x, raw[2 * i + 1].y, raw[2 * i + 1].z, raw[2 * i + 1].w};
        return __builtin_amdgcn_perm(b[j >> 1], a[j >> 1], sel);
      };
      *reinterpret_cast<uint4*>(to + TL::at(dims0 + j, octet)) = make_uint4(word(0), word(1), word(2), word(3));
    }
  };
  // operand of one 16-token step: lane (dim 32*blk + l31, half) holds tokens 16*ks + 8*half + e
  auto operand = [&](const unsigned char* tile, int blk, int ks) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const chunk_t*>(tile + TL::at(blk * 32 + l31, 2 * ks + half)));
  };

  if (n_tiles > 0) { fetch(0); stash(0, 0); }
  if (n_tiles > 1) fetch(1);
  for (int tile = 0; tile < n_tiles; ++tile) {
    __syncthreads();                         // tile is staged; the other buffer is free
    const unsigned char* kt = gram_lds + (tile & 1) * 2 * TL::kBytes;
    const unsigned char* right = kt + (is_c ? TL::kBytes : 0);
    auto step = [&](int i) {
      const int ks = share * kSteps + i;
      const bf16x8 a = operand(kt, ib, ks);
#pragma unroll
      for (int jb = 0; jb < JB; ++jb) acc[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, operand(right, jb, ks), i == 0 ? f32x16{} : acc[jb], 0, 0, 0);
    };
    step(0);
#pragma unroll 2
    for (int i = 1; i < kSteps; ++i) step(i);
    if (kShares == 1 || tile + 1 < n_tiles) {      // d = 64: the last tile's sums stay in acc
#pragma unroll
      for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int x = 0; x < 16; ++x) total[jb][x] += acc[jb][x];
    }
    if (tile + 1 < n_tiles) stash(tile + 1, (tile + 1) & 1);
    if (tile + 2 < n_tiles) fetch(tile + 2);
  }
  if constexpr (kShares == 2) {              // the second half's tokens, through LDS; the four sums are rounded once
    __syncthreads();
    double* mine = reinterpret_cast<double*>(gram_lds) + (wave % (2 * JB)) * (JB * 16 * kWave) + lane;
    if (share == 1) {
#pragma unroll
      for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int x = 0; x < 16; ++x) mine[(jb * 16 + x) * kWave] = (double)total[jb][x] + (double)acc[jb][x];
    }
    __syncthreads();
    if (share == 1) return;
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
      for (int x = 0; x < 16; ++x) total[jb][x] = (float)((double)total[jb][x] + (double)acc[jb][x] + mine[(jb * 16 + x) * kWave]);
  }
  // accumulator register x of block jb: row 32*ib + acc_row(x, half), column 32*jb + l31
  float* out = p.part + (((size_t)h * p.n_chunks + chunk) * 2 + (is_c ? 1 : 0)) * D * D;
#pragma unroll
  for (int jb = 0; jb < JB; ++jb)
    if (is_c || jb <= ib) {                  // K^T K is symmetric: the blocks up to the diagonal
#pragma unroll
      for (int x = 0; x < 16; ++x) out[(size_t)(32 * ib + acc_row(x, half)) * D + 32 * jb + l31] = total[jb][x];
    }
}

// fp32 inputs: the same products on the fp32 matrix instructions, whose operands (one element per
// lane: 32 dims of one token, two tokens side by side) come straight out of [token][dim] tiles
template <int D>
__global__ __launch_bounds__(kCalThreads) void gram_f32_kernel(CalParams p) {
  constexpr int kTok = 16;                           // tokens per tile
  constexpr int kStride = D + 32;                    // the two tokens of an operand read lie 32 banks apart
  constexpr int JB = D / 32;
  constexpr bool kBoth = (JB == 4);
  __shared__ __align__(16) float kt[kTok * kStride], vt[kTok * kStride];
  const int h = blockIdx.y, chunk = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l31 = lane & 31, half = lane >> 5;
  const int ib = kBoth ? wave : (wave % JB);
  const bool do_g = kBoth || wave < JB, do_c = kBoth || wave >= JB;
  const float* k_head = reinterpret_cast<const float*>(p.k) + (int64_t)h * p.k_sh;
  const float* v_head = reinterpret_cast<const float*>(p.v) + (int64_t)h * p.v_sh;
  const int c_begin = chunk * p.tokens_per_chunk;
  const int c_end = min(p.m, c_begin + p.tokens_per_chunk);
  f32x16 accg[JB], accc[JB];
#pragma unroll
  for (int jb = 0; jb < JB; ++jb)
#pragma unroll
    for (int x = 0; x < 16; ++x) { accg[jb][x] = 0.f; accc[jb][x] = 0.f; }
  constexpr int kPieces = kTok * D / 4 / kCalThreads;
  uint4 kr[kPieces], vr[kPieces];
  auto fetch = [&](int t0) {
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
      const int i = threadIdx.x + u * kCalThreads, t = min(t0 + i / (D / 4), p.m - 1), c = (i % (D / 4)) * 4;
      kr[u] = load_chunk(k_head + (int64_t)t * p.k_st + c);
      vr[u] = load_chunk(v_head + (int64_t)t * p.v_st + c);
    }
  };
  if (c_begin < c_end) fetch(c_begin);
  for (int t0 = c_begin; t0 < c_end; t0 += kTok) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
      const int i = threadIdx.x + u * kCalThreads, r = i / (D / 4), c = (i % (D / 4)) * 4;
      const bool live = t0 + r < c_end;
      *reinterpret_cast<uint4*>(kt + r * kStride + c) = live ? kr[u] : make_uint4(0, 0, 0, 0);
      *reinterpret_cast<uint4*>(vt + r * kStride + c) = live ? vr[u] : make_uint4(0, 0, 0, 0);
    }
    __syncthreads();
    if (t0 + kTok < c_end) fetch(t0 + kTok);
#pragma unroll 4
    for (int ks = 0; ks < kTok / 2; ++ks) {
      const float* kp = kt + (2 * ks + half) * kStride + l31;
      const float* vp = vt + (2 * ks + half) * kStride + l31;
      const float a = kp[ib * 32];
#pragma unroll
      for (int jb = 0; jb < JB; ++jb) {
        if (do_g) accg[jb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, kp[jb * 32], accg[jb], 0, 0, 0);
        if (do_c) accc[jb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, vp[jb * 32], accc[jb], 0, 0, 0);
      }
    }
  }
  float* out = p.part + ((size_t)h * p.n_chunks + chunk) * 2 * D * D;
#pragma unroll
  for (int jb = 0; jb < JB; ++jb)
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const size_t at = (size_t)(32 * ib + acc_row(x, half)) * D + 32 * jb + l31;
      if (do_g && jb <= ib) out[at] = accg[jb][x];
      if (do_c) out[(size_t)D * D + at] = accc[jb][x];
    }
}

// Chunk partials -> fp64 sums in 16 x 16 tiles, the order solve_kernel keeps them in LDS: tile (i, j),
// j <= i, of K^T K, then tile (r, j) of (K^T V)^T.  Grid (tiles, heads).  A wave takes a quarter of the chunks, a lane four
// elements side by side in all of them, requested at once; the quarters meet in LDS, in order.  Bound: the partials, 27 MB
// at 65536 tokens x 8 heads, in 7.4 us.  (One
// workgroup per head summing all of it took most of the solve's 0.9 ms at 65536 tokens.)
template <int D>
__global__ __launch_bounds__(256) void gram_reduce_kernel(CalParams p) {
  constexpr int NB = D / 16, kTri = NB * (NB + 1) / 2, U = (kCalMaxChunks + 3) / 4;
  __shared__ __align__(16) f64x4 shares[3][kWave];
  const int h = blockIdx.y, tile = blockIdx.x;
  const int lane = threadIdx.x & 63, quarter = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), r = lane >> 2, c = (lane & 3) * 4;
  const bool transposed = tile >= kTri;
  size_t at;
  if (!transposed) {
    int i = 0;
    while ((i + 1) * (i + 2) / 2 <= tile) ++i;
    const int j = tile - i * (i + 1) / 2;
    at = (size_t)(16 * i + r) * D + 16 * j + c;
  } else {
    const int t = tile - kTri, cb = t / NB, j = t % NB;           // rows 16 j .. of K^T V, columns 16 cb ..
    at = (size_t)D * D + (size_t)(16 * j + r) * D + 16 * cb + c;
  }
  const float* part = p.part + (size_t)h * p.n_chunks * 2 * D * D + at;
  const int per = (p.n_chunks + 3) / 4, c0 = quarter * per, c1 = min(p.n_chunks, c0 + per);      // per <= U
  f32x4 x[U];
#pragma unroll
  for (int u = 0; u < U; ++u) x[u] = *reinterpret_cast<const f32x4*>(part + (size_t)min(c0 + u, p.n_chunks - 1) * 2 * D * D);
  f64x4 s = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (c0 + u < c1) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s[e] += (double)x[u][e];
    }
  if (quarter > 0) shares[quarter - 1][lane] = s;
  __syncthreads();
  if (quarter > 0) return;
#pragma unroll
  for (int q = 0; q < 3; ++q) s += shares[q][lane];
  double* out = p.sums + ((size_t)h * (kTri + NB * NB) + tile) * 256;
#pragma unroll
  for (int e = 0; e < 4; ++e) out[transposed ? (c + e) * 16 + r : r * 16 + c + e] = s[e];
}

// fp64 on the matrix cores, C + A B.  16x16x4: lane (l15, l4) = (lane & 15, lane >> 4) holds A[l15][l4], B[l4][l15]
// and C[4 v + l4][l15] in register v, so register v of a C is the B operand that four of its rows make, and the A operand of
// the same rows of its transpose.  4x4x4, four blocks: as if A had 4 rows, which every group of four lanes holds; C is one register.
constexpr int kLdt = 18;                      // doubles between rows of a tile: operand reads of 16 rows hit distinct banks
constexpr int kTileDoubles = 16 * kLdt;

__device__ __forceinline__ double readlane_f64(double x, int lane) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, lane), hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
}

__device__ __forceinline__ f64x4 mfma_f64(double a, double b, const f64x4& c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ __forceinline__ double mfma4_f64(double a, double b, double c) { return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0); }

// of every 16 lanes, lanes 4 Q .. 4 Q + 3 in all four groups of four
template <int Q> __device__ __forceinline__ double spread4(double x) {
  const unsigned long long bits = __builtin_bit_cast(unsigned long long, x);
  auto half = [](int w) VEC_INLINE {
    int out = w;                                // row_ror:n takes from n lanes below; the last mask names the group written
    if constexpr (Q != 0) out = __builtin_amdgcn_update_dpp(out, w, 0x120 + 4 * ((0 - Q) & 3), 0xf, 1, false);
    if constexpr (Q != 1) out = __builtin_amdgcn_update_dpp(out, w, 0x120 + 4 * ((1 - Q) & 3), 0xf, 2, false);
    if constexpr (Q != 2) out = __builtin_amdgcn_update_dpp(out, w, 0x120 + 4 * ((2 - Q) & 3), 0xf, 4, false);
    if constexpr (Q != 3) out = __builtin_amdgcn_update_dpp(out, w, 0x120 + 4 * ((3 - Q) & 3), 0xf, 8, false);
    return (uint32_t)out;
  };
  const uint32_t lo = half((int)(uint32_t)bits), hi = half((int)(uint32_t)(bits >> 32));
  return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
}

// 1 / sqrt(x) and 1 / x: the hardware's estimate (good to about 2^-24) and one step of third order
__device__ __forceinline__ double inverse_sqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}
__device__ __forceinline__ double inverse(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// Cholesky of a 16 x 16 diagonal tile by one wave: the inverse of its factor (zeros above the diagonal) goes to `tile`.
// The tile is A - X X^T, with A whole as an accumulator and X^T as one.  A pivot that is not positive marks the head.
// Four columns at a time: every lane factors the 4 x 4 block on the diagonal and inverts the factor (T; the chain from pivot
// to pivot is the square-root-free one), and the matrix cores do the rest: the four columns of the factor are
// P = A_b T^t, formed as T A_b^t because that comes out as an operand again (A is symmetric: A_b^t is register b),
// then the rows below lose P P^t; of the inverse, rows b become T times what stands there and the rows below lose
// P times that.  All in 4x4x4 instructions, a quarter of a 16x16x4 each: what the next block waits for is two of them.
// A wave alone issues an instruction about every six cycles, so their number counts as well as the chain: some 500 a tile,
// 3200 cycles (28 % more with a square root per pivot and sixteen spreads for X X^T).  A column at a time, every
// element of the pivot row broadcast by readlane to the tile and the inverse: 52 us for the solve, against 23.
// Columns of `a` left of block b are never read again.
__device__ __forceinline__ void factor_invert_tile(f64x4 a, const f64x4& xt, double* tile, int* bad) {
  const int lane = threadIdx.x & 63, l15 = lane & 15, l4 = lane >> 4, l3 = lane & 3;
  f64x4 inv;
#pragma unroll
  for (int v = 0; v < 4; ++v) inv[v] = (4 * v + l4 == l15) ? 1.0 : 0.0;
  auto each_row_block = [&](auto f) VEC_INLINE {
    f(std::integral_constant<int, 0>{}); f(std::integral_constant<int, 1>{});
    f(std::integral_constant<int, 2>{}); f(std::integral_constant<int, 3>{});
  };
  // (as 4x4x4 instructions too this is more, not less: sixteen spreads)
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) a = mfma_f64(-xt[kk], xt[kk], a);
  // a choice by bits: of ?: the compiler makes branches, with the arithmetic moved into them
  auto pick = [](uint32_t yes, double x, double y) VEC_INLINE {
    const unsigned long long xb = __builtin_bit_cast(unsigned long long, x), yb = __builtin_bit_cast(unsigned long long, y);
    const uint32_t lo = (yes & (uint32_t)xb) | (~yes & (uint32_t)yb), hi = (yes & (uint32_t)(xb >> 32)) | (~yes & (uint32_t)(yb >> 32));
    return __builtin_bit_cast(double, (unsigned long long)lo | ((unsigned long long)hi << 32));
  };
  uint32_t is0 = l3 == 0 ? ~0u : 0u, is1 = l3 == 1 ? ~0u : 0u, is2 = l3 == 2 ? ~0u : 0u;
  asm volatile("" : "+v"(is0), "+v"(is1), "+v"(is2));
  bool ok = true;
  each_row_block([&](auto bv) VEC_INLINE {
    constexpr int b = decltype(bv)::value;
    double u[4][4], m[4][4], t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) u[i][j] = readlane_f64(a[b], 16 * i + 4 * b + j);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (k < 3) {
        const double r = inverse(u[k][k]);
#pragma unroll
        for (int i = k + 1; i < 4; ++i) {
          m[i][k] = u[i][k] * r;
#pragma unroll
          for (int j = k + 1; j <= i; ++j) u[i][j] = fma(-(u[i][k] * u[j][k]), r, u[i][j]);
        }
      }
      // column l4 of the unit factor's inverse, a row at a time
      t[k] = (l4 == k) ? 1.0 : 0.0;
#pragma unroll
      for (int j = 0; j < k; ++j) t[k] = fma(-m[k][j], t[j], t[k]);
    }
    // this lane's row of T: one square root for all four
    const double row = pick(is0, t[0], pick(is1, t[1], pick(is2, t[2], t[3])));
    const double pivot = pick(is0, u[0][0], pick(is1, u[1][1], pick(is2, u[2][2], u[3][3])));
    ok &= pivot > 0.0;
    const double T = row * inverse_sqrt(pivot);
    const double P = mfma4_f64(T, a[b], 0.0);                  // P[l15][l4]
    const double minus_p = -P;
    double below[4];
    each_row_block([&](auto v) VEC_INLINE {
      constexpr int V = decltype(v)::value;
      if constexpr (V > b) {
        below[V] = spread4<V>(minus_p);
        a[V] = mfma4_f64(below[V], P, a[V]);
      }
    });
    inv[b] = mfma4_f64(T, inv[b], 0.0);
#pragma unroll
    for (int v = b + 1; v < 4; ++v) inv[v] = mfma4_f64(below[v], inv[b], inv[v]);
  });
  if (!ok) *bad = 1;
#pragma unroll
  for (int v = 0; v < 4; ++v) tile[(4 * v + l4) * kLdt + l15] = inv[v];
}

// (K^T K) W = K^T V for 16 columns of W.  Grid (d / 16, heads), eight waves; every workgroup factors
// its head's matrix itself (the factorisation is a chain of d / 16 steps that another workgroup could not
// shorten).  Everything lies in LDS as 16 x 16 fp64 tiles and every product is a v_mfma_f64_16x16x4:
//   right-looking blocked Cholesky: the diagonal tile is factored and its factor inverted by one wave,
//   the tiles below it are multiplied by that inverse, the tiles right of it lose their products.
//   The first wave keeps the chain in its registers: the tile below the diagonal comes out of its product as the
//   operands that the next diagonal tile's update takes, and that tile is factored while the others update the rest.
//   The right-hand sides ride along as one more block row, (K^T V)^T: after step s its tile s holds the
//   forward solution.  For the backward substitution wave j takes rows 16 j .. of it into registers, and
//   a solved block goes to the waves above through LDS.
// Bound: the chain of 4 x 4 blocks.  23 us for d = 128, eight heads (cycles: 30000 in the diagonal tiles, 7000 in the tiles
// below them, 7500 in the backward substitution; the other tiles' updates are waited for in the second step alone).
// Reading the next tile's operands ahead of a tile's products made the updates slower (6500 cycles against 5200 in
// that step); L_ss^-1 L_sj formed by the idle waves while the tiles below the diagonal are multiplied, so that the backward
// substitution waits for half as many products, lengthened those steps by more than it saved (the fit 0.6 us longer).
// One workgroup per head with a thread per row and plain loops took 934 us (the sums included).
template <typename T, int D>
__global__ __launch_bounds__(512) void solve_kernel(CalParams p) {
  constexpr int NB = D / 16, kTri = NB * (NB + 1) / 2, NW = 512 / kWave;
  static_assert(NB <= NW, "a wave per tile of a block column");
  extern __shared__ __align__(16) double cal_tiles[];        // [kTri + NB][kTileDoubles]
  __shared__ int bad;
  const int h = blockIdx.y, cb = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), l15 = lane & 15, l4 = lane >> 4;
  auto tile = [&](int i, int j) { return cal_tiles + (i * (i + 1) / 2 + j) * kTileDoubles; };   // row NB: the right-hand sides
  const double* src = p.sums + (size_t)h * (kTri + NB * NB) * 256;
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
  f64x4 diag = zero, xt = zero;                                // the next diagonal tile and what it loses, in the first wave
  if (wave == 0) {
    if (lane == 0) bad = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) diag[v] = src[(4 * v + l4) * 16 + l15];
  } else {
    // the other tiles, while the first wave factors: 16-byte pairs, all requested at once
    constexpr int kThreads = 512 - kWave, kPairs = (kTri + NB - 1) * 128, kTrips = (kPairs + kThreads - 1) / kThreads;
    double2 x[kTrips];
#pragma unroll
    for (int u = 0; u < kTrips; ++u) {
      const int o = 128 + min((int)threadIdx.x - kWave + u * kThreads, kPairs - 1), t = o >> 7;
      x[u] = *reinterpret_cast<const double2*>(src + (size_t)(t < kTri ? t : kTri + cb * NB + (t - kTri)) * 256 + (o & 127) * 2);
    }
#pragma unroll
    for (int u = 0; u < kTrips; ++u) {
      const int n = (int)threadIdx.x - kWave + u * kThreads, o = 128 + n, t = o >> 7, e = (o & 127) * 2;
      if (n < kPairs) *reinterpret_cast<double2*>(cal_tiles + t * kTileDoubles + (e >> 4) * kLdt + (e & 15)) = x[u];
    }
  }
  // Operands of a tile by its rows: A operands of X, B operands of X^T.  Instruction kk takes elements 4 l4 + kk of the sum,
  // whichever four they are, so that a lane reads 32 bytes in a row.
  auto by_rows = [&](const double* X) VEC_INLINE {
    const double2 x0 = *reinterpret_cast<const double2*>(X + l15 * kLdt + 4 * l4), x1 = *reinterpret_cast<const double2*>(X + l15 * kLdt + 4 * l4 + 2);
    return f64x4{x0.x, x0.y, x1.x, x1.y};
  };
  // by its columns, X[4 kk + l4][l15]: as an accumulator, or A operands of X^T
  auto by_columns = [&](const double* X) VEC_INLINE {
    f64x4 x;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) x[kk] = X[(4 * kk + l4) * kLdt + l15];
    return x;
  };
  auto products = [&](const f64x4& a, const f64x4& b, f64x4 acc) VEC_INLINE {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) acc = mfma_f64(a[kk], b[kk], acc);
    return acc;
  };
  auto wave_fence = [&]() VEC_INLINE {                         // a tile handed over inside one wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  for (int s = 0;; ++s) {
    if (wave == 0) {
      factor_invert_tile(diag, xt, tile(s, s), &bad);
    } else if (s > 0) {
      // tiles (i, j), s <= j <= i, but for the next diagonal tile, lose the products of block column s - 1
      int i = s + wave, j = s;
      while (true) {
        while (j < NB && i > NB) { ++j; i += j - (NB + 1); }
        if (j >= NB) break;
        const f64x4 c = products(-by_rows(tile(i, s - 1)), by_rows(tile(j, s - 1)), by_columns(tile(i, j)));
#pragma unroll
        for (int v = 0; v < 4; ++v) tile(i, j)[(4 * v + l4) * kLdt + l15] = c[v];
        i += NW - 1;
      }
    }
    __syncthreads();
    // below the diagonal: X = A L_ss^-T, a tile per wave, as X^T = L_ss^-1 A^T
    const int i_own = s + 1 + wave;
    if (i_own <= NB) {
      xt = products(by_rows(tile(s, s)), by_rows(tile(i_own, s)), zero);
      if (wave == 0 && s + 1 < NB) diag = by_columns(tile(s + 1, s + 1));
      wave_fence();
#pragma unroll
      for (int v = 0; v < 4; ++v) tile(i_own, s)[l15 * kLdt + 4 * v + l4] = xt[v];
    }
    __syncthreads();
    if (s + 1 == NB) break;
  }
  // L^T X = Y: X_s = L_ss^-T Y_s, then Y_j -= L_sj^T X_s for j < s.  X_s goes where Y_s^T was, register by register.
  f64x4 x = zero, lt = zero;
  if (wave < NB) {
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = tile(NB, wave)[l15 * kLdt + 4 * v + l4];
    lt = by_columns(tile(NB - 1, wave));
  }
  for (int s = NB - 1; s >= 0; --s) {
    if (wave == s) {
      x = products(lt, x, zero);
#pragma unroll
      for (int v = 0; v < 4; ++v) tile(NB, s)[v * 64 + lane] = x[v];
    }
    f64x4 lt_next = zero;
    if (wave < s) lt_next = by_columns(tile(s - 1, wave));
    __syncthreads();
    if (wave < s) {
      f64x4 solved;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) solved[kk] = tile(NB, s)[kk * 64 + lane];
      x = products(-lt, solved, x);
    }
    lt = lt_next;
  }
  // x[v]: row 16 wave + 4 v + l4 of W, column 16 cb + l15
  T* Wh = reinterpret_cast<T*>(p.W) + (size_t)h * D * D + cb * 16 + l15;
  if (wave < NB) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
      store_elem(Wh + (size_t)(16 * wave + 4 * v + l4) * D, bad ? __builtin_nanf("") : (float)x[v]);       // not positive definite: say so
  }
}

// fp64 tiles a head's sums take: K^T K up to its diagonal, and (K^T V)^T
constexpr int cal_tiles_per_head(int d) { return (d / 16) * (d / 16 + 1) / 2 + (d / 16) * (d / 16); }

// bf16: as many chunks as give each CU the one workgroup that its LDS holds, in as many rounds as it takes for no chunk to be
// longer than kCalMaxTokens (its partial sums are added in fp32, see gram_kernel) and for at least three quarters of the rounds' CUs
// to have one.  The fit, us, with chunks per head x their tokens:
//   8 heads x 42443: 31 x 1408 (0.97 rounds) 60, 34 x 1280 (1.06) 78, 56 x 768 (1.75) 72; 8 x 12000: 32 x 384 (1.00) 43, 47 x 256 50
//   48 x 8192: 5 x 1664 (0.94) 87, 6 x 1408 (1.12) 104; 96 x 4096: 2 x 2048 (0.75) 114, 3 x 1408 (1.12) 128, 8 x 512 (3.00) 145
//   65 x 2100: 3 x 768 (0.76) 90, 4 x 640 (1.02) 102, 5 x 512 (1.27) 98; 65 x 16384: 8 x 2048 (2.03) 230, 11 x 1536 (2.79) 214, 16 x 1024 247
//   130 x 8192: 4 x 2048 (2.03) 276, 5 x 1664 (2.54) 259, 8 x 1024 (4.06) 287; 300 x 2048: 1 x 2048 (1.17) 336, 2 x 1024 (2.34) 332
//   d = 64: 65 x 8192: 4 x 2048 (1.02) 52, 7 x 1280 (1.78) 45, 8 x 1024 (2.03) 51; 130 x 2088: 2 x 1280 (1.02) 49, 3 x 768 (1.52) 44
// With two workgroups of half the size on a CU and chunks of 1024 tokens: 8 x 42443 75, 32 x 16384 100 (now 92), 65 x 16384 236 (214),
// 96 x 16384 297 (271), 130 x 32768 722 (639).
// fp32: 1024 tokens per chunk, shorter ones while that leaves CUs without a workgroup (a chunk's tiles are a
// chain, and shorter chunks only tighten the fp32 sums).  Both: longer ones past 64 chunks, none shorter than 256 tokens.
void calibrate_chunks(const vector_shape& s, int& tokens_per_chunk, int& n_chunks) {
  const int m = s.seq_len, heads = s.n_kv_heads;
  int tile = kCalTile;
  if (s.dtype == VECTOR_BF16) {
    if (s.head_dim == 64) tile = 2 * kCalTile;
    const int most = (m + kCalMinTokens - 1) / kCalMinTokens, least = std::min(kCalMaxChunks, (m + kCalMaxTokens - 1) / kCalMaxTokens);
    int64_t rounds = ((int64_t)least * heads + kCalCus - 1) / kCalCus;
    do n_chunks = (int)(kCalCus * rounds / heads);
    while (4 * (int64_t)n_chunks * heads < 3 * kCalCus * rounds++);
    if (n_chunks > most) n_chunks = most;
  } else {
    int want = 1024;
    while (want > kCalMinTokens && (int64_t)((m + want - 1) / want) * heads < kCalCus) want >>= 1;
    n_chunks = (m + want - 1) / want;
  }
  if (n_chunks > kCalMaxChunks) n_chunks = kCalMaxChunks;
  if (n_chunks < 1) n_chunks = 1;
  tokens_per_chunk = ((m + n_chunks - 1) / n_chunks + tile - 1) / tile * tile;
  n_chunks = (m + tokens_per_chunk - 1) / tokens_per_chunk;
  if (n_chunks < 1) n_chunks = 1;
}

template <typename T, int D>
int run_calibrate(const vector_shape& s, CalParams& p, hipStream_t stream) {
  const dim3 grid(p.n_chunks, s.n_kv_heads);
  if constexpr (Elem<T>::kDtype == VECTOR_BF16) {
    constexpr size_t lds = 4 * GramTile<D>::kBytes;
    VEC_HIP(set_max_lds(reinterpret_cast<const void*>(gram_kernel<D>), lds));
    hipLaunchKernelGGL(gram_kernel<D>, grid, dim3(kGramThreads), lds, stream, p);
  } else {
    hipLaunchKernelGGL(gram_f32_kernel<D>, grid, dim3(kCalThreads), 0, stream, p);
  }
  hipLaunchKernelGGL(gram_reduce_kernel<D>, dim3(cal_tiles_per_head(D), s.n_kv_heads), dim3(256), 0, stream, p);
  constexpr int NB = D / 16;
  constexpr size_t lds = (size_t)(NB * (NB + 1) / 2 + NB) * kTileDoubles * sizeof(double);
  VEC_HIP(set_max_lds(reinterpret_cast<const void*>(solve_kernel<T, D>), lds));
  hipLaunchKernelGGL((solve_kernel<T, D>), dim3(NB, s.n_kv_heads), dim3(512), lds, stream, p);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

}  // namespace

size_t calibrate_workspace_bytes(const vector_shape& s) {
  int tpc, nc;
  calibrate_chunks(s, tpc, nc);
  const size_t dd = (size_t)s.head_dim * s.head_dim;
  return align_up((size_t)s.n_kv_heads * nc * 2 * dd * sizeof(float), 256) +
         align_up((size_t)s.n_kv_heads * cal_tiles_per_head(s.head_dim) * 256 * sizeof(double), 256);
}

int launch_calibrate(const vector_shape& s, const void* k, const void* v, void* W, void* ws, hipStream_t stream) {
  CalParams p;
  p.k = k; p.v = v; p.W = W; p.m = s.seq_len;
  const int D = s.head_dim;
  p.k_st = s.k_stride_tok ? s.k_stride_tok : D;
  p.k_sh = s.k_stride_head ? s.k_stride_head : (int64_t)s.seq_len * p.k_st;
  p.v_st = s.v_stride_tok ? s.v_stride_tok : D;
  p.v_sh = s.v_stride_head ? s.v_stride_head : (int64_t)s.seq_len * p.v_st;
  calibrate_chunks(s, p.tokens_per_chunk, p.n_chunks);
  const size_t dd = (size_t)D * D;
  unsigned char* w8 = reinterpret_cast<unsigned char*>(ws);
  p.part = reinterpret_cast<float*>(w8);
  w8 += align_up((size_t)s.n_kv_heads * p.n_chunks * 2 * dd * sizeof(float), 256);
  p.sums = reinterpret_cast<double*>(w8);
  if (s.dtype == VECTOR_BF16) {
    if (D == 128) return run_calibrate<bf16_t, 128>(s, p, stream);
    if (D == 64) return run_calibrate<bf16_t, 64>(s, p, stream);
  } else if (s.dtype == VECTOR_F32) {
    if (D == 128) return run_calibrate<float, 128>(s, p, stream);
    if (D == 64) return run_calibrate<float, 64>(s, p, stream);
  } else {
    return VECTOR_ERR_DTYPE;
  }
  return VECTOR_ERR_SHAPE;
}

}  // namespace vec
