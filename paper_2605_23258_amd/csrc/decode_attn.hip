// Decode attention over the packed VECTOR cache (Section 3.2, Step 3: values of
// approximated tokens are rebuilt from their keys, v_hat = k W, at generation time).
//
// One softmax runs over the live retained rows and the approximated rows together.
// Because the rebuilt value is linear in the key, sum_t p_t (k_t W) = (sum_t p_t k_t) W:
// the kernels accumulate z = sum p_t k_t over the approximated rows and apply W to that, once
// per (sequence, KV head) in the combine step or, in small launches, once per piece of approximated
// rows (APPLY), so every cache row is read exactly once and no value row is ever materialised.
//
// The path is bound by HBM (about 5 flop per byte): a row of the cache is read by
// row_bytes/16 adjacent lanes, 16 bytes each, so every load instruction of a wave covers
// 1 KiB of consecutive memory, and every cache row is read exactly once per step.
//
//   decode_split_mfma_kernel : bf16 caches.  A workgroup owns a range of rows of one segment (retained or
//                           approximated; see grid_split), or several ranges (see PlannedSplits).  Waves
//                           park 32-row tiles in LDS and run both products (scores, then
//                           weights times rows) on the matrix cores; see the comment above
//                           the kernel.  Variants: ROPE (approximated rows are un-rotated
//                           before they stand in for values), LITERAL (v_hat = k W rebuilt per
//                           row instead of the reassociated sum), PAGED, PLANNED (sequences of different
//                           lengths cut on the device), APPLY (pieces of approximated rows apply W).
//   decode_split_kernel   : fp32 caches: the same split with vector-ALU dot products (partial
//                           dot product per lane, rotate-add across the lanes of a row,
//                           online softmax per lane group).
//   decode_combine_kernel, decode_combine_few_kernel : merge the splits, apply W to z, normalise, store.
#include <type_traits>

#include "common.hpp"
#include "decode_rows.hpp"
#include "launch.hpp"

namespace vec {

namespace {

struct DecodeParams {
  const void* q; const void* k_ret; const void* v_ret; const void* k_apx; const void* W;
  const int32_t* len_retain;
  // per-sequence capacities and first rows of the sequences' blocks (all null: uniform blocks)
  const int32_t* cap_retain_seq; const int32_t* n_approx_seq;
  const int64_t* ret_row_start; const int64_t* apx_row_start;
  // the step's own token (null: none): exact key and value [B, Hkv, D]; it is attended as row
  // len_retain[b] of the retained segment and stored there when the block has room
  const void* k_new; const void* v_new;
  // paged retained segments (null: contiguous): block ids [B, Hkv, blocks_per_seq]; a block is
  // 1 << block_shift rows of the k_ret / v_ret pools
  const int32_t* block_table;
  int block_shift, blocks_per_seq;
  void* out;
  float* part;            // [B, Hkv, S, 2*G + G*D] floats: (m, l)[G], acc[G][D]
  int B, Hq, Hkv, cap_retain, n_approx;
  int splits_ret, splits_apx;   // workgroups per (sequence, head) on each segment
  int by_kind;                  // the grid is (KV head, sequence, split) and not (split, KV head, sequence)
  // Sequences of different lengths (see PlannedSplits): [B, Hkv, 2] (first partial, number of partials) of either segment; and what
  // a step of approximated rows counts in steps of retained ones
  int2* plan;
  float plan_apx;
  int plan_most_retained;       // workgroups
  int64_t w_sh;           // element stride between per-head W
  float c2;               // scale * log2(e)
  int literal;            // approximated rows: rebuild v_hat = k W per row instead of (sum p k) W
  int only_values;        // the partials of approximated rows are values already: W is not the merge's
  int out_f32;            // store the result as fp32 whatever the cache dtype
};

// Where the rows of one (sequence, KV head) lie: row offsets into k_ret / v_ret and into k_apx,
// the live length of the retained segment and the length of the approximated one.
struct SegmentRows {
  size_t ret_row0, apx_row0;
  int len_retain, n_approx, new_row, cap;
  const int32_t* blocks;      // paged: this (sequence, head)'s block ids; ret_row0 is then 0
  int block_shift;
};
// row r of the retained segment as a row of the k_ret / v_ret arrays.  PAGED is a template
// argument of the kernels: the lookups cost registers that the contiguous layout should not pay.
template <bool PAGED>
__device__ __forceinline__ size_t retained_row(const SegmentRows& s, int r) {
  if (PAGED) return ((size_t)s.blocks[r >> s.block_shift] << s.block_shift) + (size_t)(r & ((1 << s.block_shift) - 1));
  return s.ret_row0 + (size_t)r;
}
// of a sequence with the capacity, approximated rows, live retained rows and first rows given
__device__ __forceinline__ SegmentRows sequence_rows(const DecodeParams& p, int b, int h, int cap, int n_approx, int live, int64_t ret0, int64_t apx0) {
  SegmentRows s;
  s.n_approx = n_approx;
  s.ret_row0 = (size_t)ret0 + (size_t)h * cap;
  s.apx_row0 = (size_t)apx0 + (size_t)h * n_approx;
  s.blocks = nullptr;
  s.block_shift = 0;
  if (p.block_table) {
    s.blocks = p.block_table + ((size_t)b * p.Hkv + h) * p.blocks_per_seq;
    s.block_shift = p.block_shift;
    s.ret_row0 = 0;
  }
  s.len_retain = live;
  s.cap = cap;
  s.new_row = -1;
  if (p.k_new) { s.new_row = s.len_retain; s.len_retain += 1; }      // the new token is the last live row
  return s;
}
__device__ __forceinline__ SegmentRows segment_rows(const DecodeParams& p, int b, int h) {
  int cap = p.cap_retain, n_approx = p.n_approx;
  int64_t ret0 = (int64_t)b * p.Hkv * cap, apx0 = (int64_t)b * p.Hkv * n_approx;
  if (p.cap_retain_seq) {
    cap = max(p.cap_retain_seq[b], 0);
    n_approx = max(p.n_approx_seq[b], 0);
    ret0 = p.ret_row_start[b];
    apx0 = p.apx_row_start[b];
  }
  return sequence_rows(p, b, h, cap, n_approx, min(max(p.len_retain[b], 0), cap), ret0, apx0);
}

constexpr int DT_ = 256;          // threads per workgroup
constexpr int DW = DT_ / kWave;   // waves
constexpr int kUnroll = 4;        // rows per lane group in flight

// Rows of one segment of one (sequence, KV head) that a workgroup takes
struct SplitRows {
  int b, h;
  bool is_apx;
  int begin, end;
  size_t slot;                    // of the partial
  SegmentRows seg;
};
// One range per workgroup, the grid says which: as many splits for every sequence.  Ranges are multiples of STEP rows, so
// that loads stay aligned to it.
template <int STEP> __device__ __forceinline__ SplitRows grid_split(const DecodeParams& p) {
  SplitRows r;
  const int split = p.by_kind ? blockIdx.z : blockIdx.x;
  r.h = p.by_kind ? blockIdx.x : blockIdx.y;
  r.b = p.by_kind ? blockIdx.y : blockIdx.z;
  r.seg = segment_rows(p, r.b, r.h);
  r.is_apx = split >= p.splits_ret;
  const int len = r.is_apx ? r.seg.n_approx : r.seg.len_retain;
  const int n_sp = r.is_apx ? p.splits_apx : p.splits_ret, sp = r.is_apx ? split - p.splits_ret : split;
  const int steps = (len + STEP - 1) / STEP;
  r.begin = (int)((int64_t)steps * sp / n_sp) * STEP;
  r.end = min(len, (int)((int64_t)steps * (sp + 1) / n_sp) * STEP);
  r.slot = ((size_t)r.b * p.Hkv + r.h) * (p.splits_ret + p.splits_apx) + split;
  return r;
}

// Sequences of different lengths: the same share of the work for every workgroup, wherever one sequence's rows end and
// the next one's begin.  With as many splits for every sequence the longest are waited for.  The host does not know the live lengths;
// every workgroup adds the work up itself, lane b that of sequence b.  The retained rows are one line, sequence after
// sequence, head after head, and the approximated rows another; the first workgroups share the first, the others the second, so
// that a CU, which gets two workgroups half a grid apart, has one of each (all of both lines in one, 32 sequences of up to
// 32768 tokens 89 us, now 86; 16 of them 52.5, 48.6).  A workgroup takes the granules that begin in its share; the arithmetic is in
// decode_rows.hpp.  The workgroup with a segment's first granule says in `plan` where its partials begin and how many there are.
//   A step, us, as many splits for every sequence / this: 24 sequences of 4000 to 16000 tokens on rotated keys 51.5 / 44.6, plain 43.1 /
//   40.4; 16 of 8192 to 32768 62.2 / 52.2, plain 55.2 / 48.6.
struct PlannedSequence { int cap, n_approx, live; long long ret0, apx0; };
struct PlannedSplits {
  const DecodeParams& p;
  int id, share, lo, hi, log_rows;           // a granule is 1 << log_rows rows
  int b, h, at;                              // the segment at hand begins at `at`
  bool is_apx, done;
  PlannedSequence s;                         // sequence b
  // Scalars are kept scalar: the compiler would keep in vector registers what follows from a float or from memory.
  static __device__ __forceinline__ int same(int x) { return __builtin_amdgcn_readfirstlane(x); }
  static __device__ __forceinline__ long long same(long long x) { return ((long long)same((int)(x >> 32)) << 32) | (uint32_t)same((int)x); }
  __device__ __forceinline__ int granules(int len) const { return plan_granules(len, log_rows); }
  // of a sequence with nothing cached an empty granule, whose workgroup writes the empty partial
  __device__ __forceinline__ int granules_ret(const PlannedSequence& x) const {
    const int n = granules(x.live + (p.k_new ? 1 : 0));
    return x.n_approx == 0 ? max(n, 1) : n;
  }
  static __device__ __forceinline__ PlannedSequence sequence(const DecodeParams& p, int i) {
    const int cap = planned_rows(p.cap_retain, p.cap_retain_seq[i]);
    return {cap, planned_rows(p.n_approx, p.n_approx_seq[i]), min(max(p.len_retain[i], 0), cap), p.ret_row_start[i], p.apx_row_start[i]};
  }
  __device__ __forceinline__ explicit PlannedSplits(const DecodeParams& p_) : p(p_) {
    const int lane = threadIdx.x & 63;
    const PlannedSequence x = sequence(p, min(lane, p.B - 1));
    // granules so long that a line stays shorter than kMaxPlanUnits: 32 rows unless the cache were larger than the memory
    log_rows = kLogGranule;
    int len_r = plan_length(granules_ret(x)), len_a = plan_length(granules(x.n_approx));
    float top_r = wave_max_dpp((float)len_r), top_a = wave_max_dpp((float)len_a);
    while (__builtin_expect(plan_too_long(fmaxf(top_r, top_a), p.B, p.Hkv, log_rows), 0)) {
      log_rows = same(log_rows + 1);
      len_r = plan_length(granules_ret(x));
      len_a = plan_length(granules(x.n_approx));
      top_r = wave_max_dpp((float)len_r);
      top_a = wave_max_dpp((float)len_a);
    }
    const int seq_r = lane < p.B ? len_r * p.Hkv : 0, seq_a = lane < p.B ? len_a * p.Hkv : 0;
    const int upto_r = wave_incl_scan_dpp(seq_r), upto_a = wave_incl_scan_dpp(seq_a);
    const int total_r = __builtin_amdgcn_readlane(upto_r, 63), total_a = __builtin_amdgcn_readlane(upto_a, 63), wgs = gridDim.x;
    const int wgs_r = same(plan_retained(wgs, p.plan_most_retained, total_r, total_a, __builtin_amdgcn_rcpf((float)total_r + (float)total_a * p.plan_apx)));
    id = blockIdx.x;
    is_apx = id >= wgs_r;
    const int mine = is_apx ? id - wgs_r : id, total = is_apx ? total_a : total_r;
    share = same(plan_share(total, is_apx ? top_a : top_r, __builtin_amdgcn_rcpf((float)(is_apx ? wgs - wgs_r : wgs_r))));
    lo = mine * share;
    hi = lo + share;
    done = lo >= total;                      // of small caches fewer workgroups than the grid has
    b = h = at = 0;
    s = PlannedSequence{};
    if (done) return;
    const int upto = is_apx ? upto_a : upto_r, of_sequence = is_apx ? seq_a : seq_r;
    b = __popcll(__ballot(upto <= lo));
    at = __builtin_amdgcn_readlane(upto - of_sequence, b);
    const int head = __builtin_amdgcn_readlane(is_apx ? len_a : len_r, b);
    h = same(plan_head(lo - at, head, __builtin_amdgcn_rcpf((float)head)));
    at += h * head;
    auto of_b = [&](int v) VEC_INLINE { return __builtin_amdgcn_readlane(v, b); };
    auto of_b64 = [&](long long v) VEC_INLINE { return ((long long)of_b((int)(v >> 32)) << 32) | (uint32_t)of_b((int)v); };
    s = {of_b(x.cap), of_b(x.n_approx), of_b(x.live), of_b64(x.ret0), of_b64(x.apx0)};
  }
  // the next rows of this workgroup; false: there are none
  __device__ __forceinline__ bool next(SplitRows& r) {
    while (!done) {
      const int n_r = granules_ret(s), n_a = granules(s.n_approx), n = is_apx ? n_a : n_r;
      const PlanPiece piece = plan_piece(at, n, lo, share);
      const int pair = b * p.Hkv + h, place = plan_place(id, pair, is_apx, p.B * p.Hkv);
      const bool any = piece.first < piece.last;
      if (any) {
        r.b = b; r.h = h; r.is_apx = is_apx;
        r.seg = sequence_rows(p, b, h, s.cap, s.n_approx, s.live, s.ret0, s.apx0);
        r.begin = piece.first << log_rows;
        r.end = (int)min((int64_t)(is_apx ? r.seg.n_approx : r.seg.len_retain), (int64_t)piece.last << log_rows);
        r.slot = (size_t)place;
        if (piece.first == 0 && threadIdx.x == 0) {
          p.plan[2 * pair + (is_apx ? 1 : 0)] = make_int2(place, plan_partials(at, n, lo, share));
          if ((is_apx ? n_r : n_a) == 0) p.plan[2 * pair + (is_apx ? 0 : 1)] = make_int2(0, 0);
        }
      }
      at += plan_length(n);
      done = at >= hi;
      if (++h == p.Hkv) {
        h = 0;
        if (++b == p.B) done = true;
        if (!done) {
          const PlannedSequence x = sequence(p, b);
          s = {same(x.cap), same(x.n_approx), same(x.live), same(x.ret0), same(x.apx0)};
        }
      }
      if (any) return true;
    }
    return false;
  }
};

// what a workgroup of a split launch does
template <int STEP, bool PLANNED, typename F> __device__ __forceinline__ void for_split_rows(const DecodeParams& p, F attend) {
  if constexpr (PLANNED) {
    static_assert(STEP == kStepGranules << kLogGranule, "a step of the bf16 kernel");
    PlannedSplits splits(p);
    SplitRows r;
    while (splits.next(r)) {
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));                  // what is made of it would be kept in registers from range to range
      attend(r, tid);
      __syncthreads();                               // LDS may be written again
    }
  } else {
    attend(grid_split<STEP>(p), (int)threadIdx.x);
  }
}

// The workgroup whose rows include the step's own token stores it in the cache (when the block has
// room) for the steps to come; this step reads it from the caller's buffers, so nothing waits for
// the store.
template <typename T, int D, bool PAGED>
__device__ __forceinline__ void append_new_row(const DecodeParams& p, const SegmentRows& seg, bool is_apx, int row_begin, int row_end,
                                               const T* k_new, const T* v_new, int tid) {
  constexpr int kPieces = D * (int)sizeof(T) / 16;
  if (is_apx || seg.new_row < row_begin || seg.new_row >= row_end || seg.new_row >= seg.cap) return;
  if (tid < 2 * kPieces) {
    const int piece = tid % kPieces;
    const bool is_v = tid >= kPieces;
    unsigned char* dst = reinterpret_cast<unsigned char*>(const_cast<void*>(is_v ? p.v_ret : p.k_ret)) +
                         retained_row<PAGED>(seg, seg.new_row) * D * sizeof(T) + piece * 16;
    const unsigned char* src = reinterpret_cast<const unsigned char*>(is_v ? v_new : k_new) + piece * 16;
    *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
  }
}

// sum over the LPR adjacent lanes that share a row; every lane of the group gets the total
template <int LPR> __device__ __forceinline__ float group_sum(float x) {
  if constexpr (LPR == 16) {
    // rotate-add inside a DPP row of 16 lanes: no LDS traffic
#define VEC_ROR_ADD(n) x += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x120 + (n), 0xf, 0xf, false))
    VEC_ROR_ADD(8); VEC_ROR_ADD(4); VEC_ROR_ADD(2); VEC_ROR_ADD(1);
#undef VEC_ROR_ADD
    return x;
  } else {
#pragma unroll
    for (int o = LPR / 2; o >= 1; o >>= 1) x += __shfl_xor(x, o, kWave);
    return x;
  }
}

// ROPE: the cache holds keys after their rotary embedding; logits use them as cached, and the rows
// that stand in for values of approximated tokens are the keys turned back by their original
// positions (rp.positions, one per row of k_apx).
template <typename T, int D, int G, bool PAGED, bool ROPE>
__device__ __forceinline__ void attend_rows(const DecodeParams& p, const RopeParams& rp, const SplitRows& range, int tid) {
  constexpr int E = Elem<T>::kPerChunk;          // elements per 16-byte piece
  constexpr int LPR = D / E;                     // lanes per row
  constexpr int RPI = kWave / LPR;               // rows per wave-wide load instruction
  constexpr int PSZ = 2 * G + G * D;

  __shared__ float ml_lds[DW][2][G];
  __shared__ float red_lds[DW][G][D];

  constexpr int kStepRows = DW * RPI * kUnroll;
  const int h = range.h, b = range.b;
  const int lane = tid & 63, wave = tid >> 6;
  const int grp = lane / LPR, piece = lane % LPR;
  const SegmentRows seg = range.seg;
  const bool is_apx = range.is_apx;
  const int seg_len = is_apx ? seg.n_approx : seg.len_retain;
  const int row_begin = range.begin, row_end = range.end;

  const size_t bh = (size_t)b * p.Hkv + h;
  // a segment's rows: the approximated block, the retained block, or (paged) the retained pool
  const T* kseg = is_apx ? reinterpret_cast<const T*>(p.k_apx) + seg.apx_row0 * D : reinterpret_cast<const T*>(p.k_ret);
  const T* vseg = reinterpret_cast<const T*>(p.v_ret);
  auto seg_row = [&](int r) { return is_apx ? (size_t)r : retained_row<PAGED>(seg, r); };
  const T* k_new = p.k_new ? reinterpret_cast<const T*>(p.k_new) + bh * D : kseg;
  const T* v_new = p.k_new ? reinterpret_cast<const T*>(p.v_new) + bh * D : vseg;
  append_new_row<T, D, PAGED>(p, seg, is_apx, row_begin, row_end, k_new, v_new, tid);

  // this lane's slice of the G query rows, pre-scaled into the log2 domain
  float qf[G][E];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint4 raw = load_chunk(reinterpret_cast<const T*>(p.q) + ((size_t)b * p.Hq + (size_t)h * G + g) * D + piece * E);
    Unpack16<T>::run(raw, qf[g]);
#pragma unroll
    for (int e = 0; e < E; ++e) qf[g][e] *= p.c2;
  }

  float m_run[G], l_run[G], acc[G][E];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    m_run[g] = -INFINITY; l_run[g] = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) acc[g][e] = 0.f;
  }

  // ROPE: the rotary pair of each of the lane's E elements, and its frequency.  Pairs (x[2i], x[2i+1])
  // lie inside the lane's piece; pairs (x[i], x[i + D/2]) are split between this lane and the lane
  // LPR/2 further along the row, which holds the same e of the other half.
  const int32_t* pos_seg = (ROPE && is_apx && rp.positions) ? rp.positions + seg.apx_row0 : nullptr;
  const bool lower_half = piece < LPR / 2;
  float t_hi[E], t_lo[E];
  if (ROPE && is_apx) {
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const int i = rp.interleaved ? (piece * E + e) / 2 : (piece % (LPR / 2)) * E + e;
      t_hi[e] = rp.turns_hi[i];
      t_lo[e] = rp.turns_lo[i];
    }
  }
  auto unrotate_row = [&](const float* kf, int pos, float* out) {
    const float pf = (float)pos;
    if (rp.interleaved) {
#pragma unroll
      for (int e = 0; e < E; e += 2) {
        float cs, sn;
        rotary_cos_sin(pf, t_hi[e], t_lo[e], cs, sn);
        rotary_back(kf[e], kf[e + 1], cs, sn, out[e], out[e + 1]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const float other = __shfl_xor(kf[e], LPR / 2, kWave);
        float cs, sn, a_pre, b_pre;
        rotary_cos_sin(pf, t_hi[e], t_lo[e], cs, sn);
        rotary_back(lower_half ? kf[e] : other, lower_half ? other : kf[e], cs, sn, a_pre, b_pre);
        out[e] = lower_half ? a_pre : b_pre;
      }
    }
  };

  // The loop bound is the same for every lane of a wave; rows past the range are masked.
  // The rows of the next step are requested before the current ones are consumed.
  auto fetch = [&](uint4* kraw, uint4* vraw, int base) {
    const int r0 = base + grp * kUnroll;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int r = min(r0 + u, seg_len - 1);      // clamped: never reads past the live rows
      const bool fresh = !is_apx && r == seg.new_row;        // the step's own token comes from the caller's buffers
      const size_t at = seg_row(fresh ? 0 : r) * D + piece * E;
      kraw[u] = load_chunk(fresh ? k_new + piece * E : kseg + at);
      if (!is_apx) vraw[u] = load_chunk(fresh ? v_new + piece * E : vseg + at);
      else if (ROPE) vraw[u].x = (uint32_t)((pos_seg ? pos_seg[r] : r) + rp.pos_offset);    // the row's position rides along
    }
  };
  auto consume = [&](const uint4* kraw, const uint4* vraw, int base) {
    const int r0 = base + grp * kUnroll;
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      float kf[E];
      Unpack16<T>::run(kraw[u], kf);
      float s[G];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) d = fmaf(qf[g][e], kf[e], d);
        s[g] = group_sum<LPR>(d);
      }
      const bool live = r0 + u < row_end;
      bool grew = false;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (!live) s[g] = -INFINITY;
        grew |= s[g] > m_run[g];
      }
      if (__any(grew)) {                             // rare once the running maxima have settled
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float m_new = fmaxf(m_run[g], s[g]);
          const float alpha = (m_new == -INFINITY) ? 1.f : fast_exp2(m_run[g] - m_new);
          l_run[g] *= alpha;
#pragma unroll
          for (int e = 0; e < E; ++e) acc[g][e] *= alpha;
          m_run[g] = m_new;
        }
      }
      float rowf[E];
      if (is_apx) {
        if (ROPE) {
          unrotate_row(kf, (int)vraw[u].x, rowf);
        } else {
#pragma unroll
          for (int e = 0; e < E; ++e) rowf[e] = kf[e];
        }
      } else {
        Unpack16<T>::run(vraw[u], rowf);
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float pg = (m_run[g] == -INFINITY) ? 0.f : fast_exp2(s[g] - m_run[g]);
        l_run[g] += pg;
#pragma unroll
        for (int e = 0; e < E; ++e) acc[g][e] = fmaf(pg, rowf[e], acc[g][e]);
      }
    }
  };
  uint4 ka[kUnroll], va[kUnroll], kb[kUnroll], vb[kUnroll];
  int base = row_begin + wave * RPI * kUnroll;
  if (base < row_end) fetch(ka, va, base);
  while (base < row_end) {
    const int b1 = base + kStepRows;
    if (b1 < row_end) fetch(kb, vb, b1);
    consume(ka, va, base);
    if (b1 >= row_end) break;
    const int b2 = b1 + kStepRows;
    if (b2 < row_end) fetch(ka, va, b2);
    consume(kb, vb, b1);
    base = b2;
  }

  // ---- merge the lane groups of a wave (each ran its own softmax), then the waves ----
#pragma unroll
  for (int o = LPR; o < kWave; o <<= 1) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float m2 = __shfl_xor(m_run[g], o, kWave), l2 = __shfl_xor(l_run[g], o, kWave);
      const float mn = fmaxf(m_run[g], m2);
      const float a = (m_run[g] == -INFINITY) ? 0.f : fast_exp2(m_run[g] - mn);
      const float c = (m2 == -INFINITY) ? 0.f : fast_exp2(m2 - mn);
      l_run[g] = l_run[g] * a + l2 * c;
#pragma unroll
      for (int e = 0; e < E; ++e) acc[g][e] = acc[g][e] * a + __shfl_xor(acc[g][e], o, kWave) * c;
      m_run[g] = mn;
    }
  }
  if (lane < LPR) {
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < E; ++e) red_lds[wave][g][piece * E + e] = acc[g][e];
  }
  if (lane == 0) {
#pragma unroll
    for (int g = 0; g < G; ++g) { ml_lds[wave][0][g] = m_run[g]; ml_lds[wave][1][g] = l_run[g]; }
  }
  __syncthreads();

  float* out = p.part + range.slot * PSZ;
  for (int i = tid; i < G * D; i += DT_) {
    const int g = i / D, j = i % D;
    float m = -INFINITY;
#pragma unroll
    for (int wv = 0; wv < DW; ++wv) m = fmaxf(m, ml_lds[wv][0][g]);
    float a = 0.f;
#pragma unroll
    for (int wv = 0; wv < DW; ++wv) {
      const float mw = ml_lds[wv][0][g];
      if (mw != -INFINITY) a += red_lds[wv][g][j] * fast_exp2(mw - m);
    }
    out[2 * G + i] = a;
  }
  if (tid < G) {
    const int g = tid;
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int wv = 0; wv < DW; ++wv) m = fmaxf(m, ml_lds[wv][0][g]);
#pragma unroll
    for (int wv = 0; wv < DW; ++wv) {
      const float mw = ml_lds[wv][0][g];
      if (mw != -INFINITY) l += ml_lds[wv][1][g] * fast_exp2(mw - m);
    }
    out[2 * g] = m;
    out[2 * g + 1] = l;
  }
}
template <typename T, int D, int G, bool PAGED = false, bool ROPE = false>
__global__ __launch_bounds__(DT_) void decode_split_kernel(DecodeParams p, RopeParams rp) {
  constexpr int kStepRows = DW * (kWave / (D / Elem<T>::kPerChunk)) * kUnroll;
  for_split_rows<kStepRows, false>(p, [&](const SplitRows& r, int tid) VEC_INLINE { attend_rows<T, D, G, PAGED, ROPE>(p, rp, r, tid); });
}

// ---------------------------------------------------------------------------
// bf16 caches: the same split, on the matrix cores.  Rows still arrive as 1 KiB
// wave-wide loads (16 bytes per lane, adjacent lanes on one row); a wave parks a tile of
// 32 rows in its own slice of LDS and reads it back in operand order:
//   scores   S[t][g] = sum_e K[t][e] q[g][e]     A = key tile (16-byte reads along a row),
//                                                 B = the G query rows, twice
//   output   O[j][g] += sum_t R[t][j] P[t][g]    A = tile of R read down its columns
//                                                 (R = values, or the keys themselves for
//                                                 approximated rows), B = P
// The accumulator layout of S (column g on lane g, sixteen tokens in the registers of a
// lane) is already the B-operand layout of the second product once the contraction index
// is numbered the way those registers number the tokens, so P never leaves its lane.  P is
// fed to the matrix core as its bf16 value (columns g) and the remainder of that rounding
// (columns G + g), which keeps the weights to about 2^-16 relative.
// ---------------------------------------------------------------------------
constexpr int kTileRows = 32;

typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;

template <int D> struct MfmaDecodeTile {
  static constexpr int kRowBytes = D * 2;
  static constexpr int kStride = kRowBytes + 16;            // LDS row stride: 16-byte reads of 32 rows hit distinct banks
  static constexpr int kPieces = kRowBytes / 16;            // 16-byte pieces per row
  static constexpr int kRowsPerLoad = kWave / kPieces;
  static constexpr int kLoads = kTileRows / kRowsPerLoad;   // wave-wide loads per tile and tensor
  static constexpr int kTileBytes = kTileRows * kStride;
  static constexpr int kTiles = DW * 2 * kTileBytes;
  static constexpr int kParts = kTiles;                     // z's three parts, where the launch applies W (APPLY)
  static constexpr int kLdsBytes = kTiles + 24 * kStride;
  // W^T's place while approximated rows stream: the value tiles, 32 rows each; the 16-byte slots of a row are permuted by the row
  static __device__ __forceinline__ uint32_t w_row(int row) { return (uint32_t)((row / kTileRows * 2 + 1) * kTileBytes + row % kTileRows * kRowBytes); }
  static __device__ __forceinline__ int w_twist(int row) { return kPieces >= 16 ? (row & 15) : ((row >> 1) & 7); }
};
// APPLY, plain rows where the launch is small (see launch_split): a piece of approximated rows leaves values, its weighted key sum times W, and the
// merge has no W to wait for.  W comes into the value tiles, which plain keys do not use, while the rows stream, and these pieces
// have half the bytes of the others.  Not with more than eight query heads, whose sums take the tiles' place; nor for rotated
// keys, where these pieces are the longer ones.
constexpr int kMostApplying = 8;

// Elements j .. j + 3 (j a multiple of 4) of a row of z, in three bf16 parts eight rows of `STRIDE` bytes apart: its 24 bits, eight at a
// time, cut and not rounded (above bf16's largest number a rounded first part would be infinite, and the second minus infinity; of an
// infinite z the first part is all).  Inside 16 contraction indices 8 a + 4 h + c in the order 8 h + 4 a + c, which is how the
// transposing read hands out W's rows.
template <int STRIDE> __device__ __forceinline__ void store_parts(unsigned char* row, int j, f32x4 z) {
  const int within = j & 15, pos = (j & ~15) + 8 * ((within >> 2) & 1) + 4 * (within >> 3);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    uint32_t top[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) top[e] = __float_as_uint(z[e]) & 0xffff0000u;
    *reinterpret_cast<uint2*>(row + q * 8 * STRIDE + pos * 2) = make_uint2(top[0] >> 16 | top[1], top[2] >> 16 | top[3]);
#pragma unroll
    for (int e = 0; e < 4; ++e) z[e] = q == 0 && (top[e] & 0x7fffffffu) == 0x7f800000u ? 0.f : z[e] - __uint_as_float(top[e]);
  }
}

// ROPE: the cached keys carry rotary position embedding.  Logits use them as cached; the
// rows that stand in for values of approximated tokens are the keys turned back by their
// original positions (rp.positions, one per row of k_apx), written to the second tile as bf16.
// LITERAL: approximated rows are rebuilt one by one, v_hat = k W, before they are weighted.
template <int D, int G, bool ROPE, bool LITERAL, bool PAGED, bool APPLY>
__device__ __forceinline__ void attend_rows_mfma(const DecodeParams& p, const RopeParams& rp, const SplitRows& range, int tid) {
  using T = bf16_t;
  using TL = MfmaDecodeTile<D>;
  constexpr int NC = D / 16;               // 16-element steps of the score contraction
  constexpr int JB = D / 32;               // 32-wide blocks of the output dimension
  constexpr int PSZ = 2 * G + G * D;
  constexpr float kNegBig = -1.0e30f;      // running maximum before any row: finite, so differences stay finite
  constexpr int kRedStride = D + 4;        // floats per row of the merge area: 16-byte writes of 2 G rows hit distinct banks
  static_assert(!APPLY || (!ROPE && !LITERAL && G <= kMostApplying), "plain rows");
  // APPLY: a wave's sums in the place of its key tile
  static_assert(DW * (2 * G * kRedStride + 2 * G) * 4 <= TL::kTiles && (!APPLY || (2 * G * kRedStride + 2 * G) * 4 <= TL::kTileBytes),
                "merge area must fit in the tile area");
  static_assert(2 * G <= 32, "weights and their remainders side by side");

  extern __shared__ __align__(16) unsigned char dec_lds[];
  // native vectors throughout: arrays of the uint4 class that are filled in one branch and used in another went to scratch
  auto load16 = [](const T* at) VEC_INLINE { return *reinterpret_cast<const u32x4*>(at); };
  auto unpack8 = [](u32x4 r, float* f) VEC_INLINE {
#pragma unroll
    for (int e = 0; e < 4; ++e) { f[2 * e] = bf16_lo(r[e]); f[2 * e + 1] = bf16_hi(r[e]); }
  };
  auto mfma = [](u32x4 a, u32x4 b, const f32x16& c) VEC_INLINE {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  };
  const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  constexpr int kStepRows = DW * kTileRows;
  const int h = range.h, b = range.b;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l31 = lane & 31, half = lane >> 5;
  const SegmentRows seg = range.seg;
  const bool is_apx = range.is_apx;
  const int seg_len = is_apx ? seg.n_approx : seg.len_retain;
  const int row_begin = range.begin, row_end = range.end;

  const size_t bh = (size_t)b * p.Hkv + h;
  // a segment's rows: the approximated block, the retained block, or (paged) the retained pool
  const T* kseg = is_apx ? reinterpret_cast<const T*>(p.k_apx) + seg.apx_row0 * D : reinterpret_cast<const T*>(p.k_ret);
  const T* vseg = reinterpret_cast<const T*>(p.v_ret);
  auto seg_row = [&](int r) { return is_apx ? (size_t)r : retained_row<PAGED>(seg, r); };
  const T* k_new = p.k_new ? reinterpret_cast<const T*>(p.k_new) + bh * D : kseg;
  const T* v_new = p.k_new ? reinterpret_cast<const T*>(p.v_new) + bh * D : vseg;
  append_new_row<T, D, PAGED>(p, seg, is_apx, row_begin, row_end, k_new, v_new, tid);

  unsigned char* k_tile = dec_lds + wave * 2 * TL::kTileBytes;
  unsigned char* v_tile = k_tile + TL::kTileBytes;
  // Rows of the second product down their columns, by the transposing LDS read: of the 16 lanes of a group, lane i hands in
  // the place of 4 consecutive columns of row i / 4 and gets the four rows of column i.
  const uint32_t r_at = lds_address((is_apx && !ROPE) ? k_tile : v_tile) + (uint32_t)((4 * half + (lane & 15) / 4) * TL::kStride +
                                                                                      (((lane >> 4) & 1) * 16 + 4 * (lane & 3)) * 2);
  const bool literal = LITERAL && is_apx;                    // rebuild every approximated value row

  // B operand of the score product: query row g on lanes g and G + g; what the columns beyond hold is never used
  const float remainder = l31 >= G ? 1.f : 0.f;
  u32x4 qf[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
    qf[c] = load16(reinterpret_cast<const T*>(p.q) + ((size_t)b * p.Hq + (size_t)h * G + l31 % G) * D + (2 * c + half) * 8);

  f32x16 o[JB];
#pragma unroll
  for (int jb = 0; jb < JB; ++jb)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[jb][v] = 0.f;
  float m_run = kNegBig, l_run = 0.f;

  const int ld_row = lane / TL::kPieces, ld_piece = lane % TL::kPieces;
  const int32_t* pos_seg = (ROPE && is_apx && rp.positions) ? rp.positions + seg.apx_row0 : nullptr;
  // Which 16 bytes of the tile a lane brings in with its i-th load.  Normally 16 adjacent lanes
  // share a row.  For approximated rows that are to be un-rotated with pairs (x[i], x[i + d/2])
  // a lane instead takes both members of its pairs: loads 2u and 2u+1 bring pieces p and
  // p + kPieces/2 of the same row, kPieces/2 adjacent lanes share a row.
  constexpr int HP = TL::kPieces / 2;
  constexpr int kRowsPerPair = kWave / HP;
  const bool paired = ROPE && is_apx && !rp.interleaved;
  const int pr_row = lane / HP, pr_piece = lane % HP;
  auto row_of = [&](int i) { return paired ? (i / 2) * kRowsPerPair + pr_row : i * TL::kRowsPerLoad + ld_row; };
  auto piece_of = [&](int i) { return paired ? pr_piece + (i & 1) * HP : ld_piece; };
  // For an approximated row under ROPE the second register set carries the row's position
  // (in .x) instead of a value row.
  // (the segment is the same for the whole workgroup: one straight-line loop per case, so that
  // all loads of a tile go out together)
  // Paged with blocks of at least a tile's 32 rows: tiles start at multiples of 32 rows, so a tile
  // lies in one block.  The block ids of the workgroup's row range sit in one register across the
  // wave (lane j: block (row_begin / block rows) + j), read once before the loop; a tile's id then
  // comes out of that register instead of memory.
  const bool tile_in_block = PAGED && !is_apx && seg.block_shift >= 5 &&
                             ((row_end - 1) >> seg.block_shift) - (row_begin >> seg.block_shift) < kWave;
  int my_block = 0;
  if (tile_in_block && row_begin < row_end) my_block = seg.blocks[block_entry(row_begin, row_end, seg.cap, seg.block_shift, lane)];
  // Rows of a tile in straight lines of loads, one line per case; the last tile of the live rows and the one with the step's
  // own token look at every row.
  const int plain_rows = is_apx || seg.new_row < 0 ? seg_len : seg.new_row;
  u32x4 kraw[TL::kLoads], vraw[TL::kLoads];
  auto fetch = [&](int base) VEC_INLINE {
    if (ROPE && is_apx) {
#pragma unroll
      for (int i = 0; i < TL::kLoads; ++i) kraw[i] = load16(kseg + (size_t)min(base + row_of(i), seg_len - 1) * D + piece_of(i) * 8);
#pragma unroll
      for (int i = 0; i < TL::kLoads; ++i) {
        const int r = min(base + row_of(i), seg_len - 1);
        vraw[i][0] = (uint32_t)((pos_seg ? pos_seg[r] : r) + rp.pos_offset);
      }
      return;
    }
    size_t tile_shift = is_apx ? 0 : seg.ret_row0;           // array row = tile_shift + segment row, where the tile is one run of rows
    if (tile_in_block) {
      const int blk = __builtin_amdgcn_readlane(my_block, (base >> seg.block_shift) - (row_begin >> seg.block_shift));
      tile_shift = ((size_t)blk << seg.block_shift) - (size_t)((base >> seg.block_shift) << seg.block_shift);
    }
    if (base + kTileRows <= plain_rows && (!PAGED || is_apx || tile_in_block)) {       // uniform
      const size_t at = (tile_shift + (size_t)base + ld_row) * D + ld_piece * 8;
#pragma unroll
      for (int i = 0; i < TL::kLoads; ++i) kraw[i] = load16(kseg + at + i * TL::kRowsPerLoad * D);
      if (!is_apx) {
#pragma unroll
        for (int i = 0; i < TL::kLoads; ++i) vraw[i] = load16(vseg + at + i * TL::kRowsPerLoad * D);
      }
      asm volatile("; tile of live rows");       // keeps the lines apart: what they have in common at their ends would be joined, through scratch
    } else if (is_apx) {
#pragma unroll
      for (int i = 0; i < TL::kLoads; ++i) kraw[i] = load16(kseg + (size_t)min(base + i * TL::kRowsPerLoad + ld_row, seg_len - 1) * D + ld_piece * 8);
      asm volatile("; last approximated rows");
    } else {
#pragma unroll
      for (int i = 0; i < TL::kLoads; ++i) {
        const int r = min(base + i * TL::kRowsPerLoad + ld_row, seg_len - 1);   // clamped: never past the live rows
        const bool fresh = r == seg.new_row;                 // the step's own token comes from the caller's buffers
        const size_t at = (tile_in_block ? tile_shift + (size_t)r : seg_row(fresh ? 0 : r)) * D + ld_piece * 8;
        kraw[i] = load16(fresh ? k_new + ld_piece * 8 : kseg + at);
        vraw[i] = load16(fresh ? v_new + ld_piece * 8 : vseg + at);
      }
      asm volatile("; last retained rows");
    }
  };
  // the lane's pieces always cover the same rotary pairs: their frequencies stay in registers
  float t_hi[8], t_lo[8];
  if (ROPE && is_apx) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int i = rp.interleaved ? (ld_piece * 8 + e) / 2 : pr_piece * 8 + e;
      t_hi[e] = rp.turns_hi[i];
      t_lo[e] = rp.turns_lo[i];
    }
  }
  auto pack8 = [](const float* f) {
    return u32x4{pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7])};
  };
  // both members of eight pairs (x[i], x[i + d/2]) of a cached key row, turned back by the row's position
  auto unrotate_pair = [&](u32x4 ra, u32x4 rb, int pos, u32x4& oa, u32x4& ob) VEC_INLINE {
    float a[8], b[8];
    const float pf = (float)pos;
    unpack8(ra, a);
    unpack8(rb, b);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float cs, sn;
      rotary_cos_sin(pf, t_hi[e], t_lo[e], cs, sn);
      rotary_back(a[e], b[e], cs, sn, a[e], b[e]);
    }
    oa = pack8(a);
    ob = pack8(b);
  };
  // pairs (x[2i], x[2i+1]): four of them inside one 16-byte piece
  auto unrotate_piece = [&](u32x4 raw, int pos) VEC_INLINE {
    float f[8];
    const float pf = (float)pos;
    unpack8(raw, f);
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      float cs, sn;
      rotary_cos_sin(pf, t_hi[e], t_lo[e], cs, sn);
      rotary_back(f[e], f[e + 1], cs, sn, f[e], f[e + 1]);
    }
    return pack8(f);
  };
  auto stage = [&]() VEC_INLINE {
    if (!is_apx || !ROPE) {
#pragma unroll
      for (int i = 0; i < TL::kLoads; ++i) *reinterpret_cast<u32x4*>(k_tile + (i * TL::kRowsPerLoad + ld_row) * TL::kStride + ld_piece * 16) = kraw[i];
      if (!is_apx) {
#pragma unroll
        for (int i = 0; i < TL::kLoads; ++i) *reinterpret_cast<u32x4*>(v_tile + (i * TL::kRowsPerLoad + ld_row) * TL::kStride + ld_piece * 16) = vraw[i];
      }
    } else {
#pragma unroll
      for (int i = 0; i < TL::kLoads; ++i) {
        const int off = row_of(i) * TL::kStride + piece_of(i) * 16;
        *reinterpret_cast<u32x4*>(k_tile + off) = kraw[i];
        if (!paired) {
          *reinterpret_cast<u32x4*>(v_tile + off) = unrotate_piece(kraw[i], (int)vraw[i][0]);
        } else if (i & 1) {
          u32x4 oa, ob;
          unrotate_pair(kraw[i - 1], kraw[i], (int)vraw[i][0], oa, ob);
          *reinterpret_cast<u32x4*>(v_tile + row_of(i - 1) * TL::kStride + piece_of(i - 1) * 16) = oa;
          *reinterpret_cast<u32x4*>(v_tile + off) = ob;
        }
      }
    }
  };
  // the tile belongs to this wave alone; these keep the compiler from moving LDS accesses of
  // different lanes across the hand-over (the hardware runs a wave's LDS operations in order)
  auto wave_fence = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };

  auto consume = [&](int base) VEC_INLINE {
    // ---- scores ----
    f32x16 s;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const u32x4 a = *reinterpret_cast<const u32x4*>(k_tile + l31 * TL::kStride + (2 * c + half) * 16);
      s = mfma(a, qf[c], c == 0 ? zero : s);
    }
    float tmax = kNegBig;
    if (base + kTileRows > row_end) {               // ragged last tile: rows past the range score -inf
#pragma unroll
      for (int v = 0; v < 16; ++v) s[v] = (base + acc_row(v, half) < row_end) ? s[v] * p.c2 : -INFINITY;
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) s[v] *= p.c2;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) tmax = fmaxf(tmax, s[v]);
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, kWave));
    if (__any(tmax > m_run)) {                       // rare once the running maxima have settled
      const float m_new = fmaxf(m_run, tmax);
      const float alpha = fast_exp2(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int jb = 0; jb < JB; ++jb)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[jb][v] *= alpha;
      m_run = m_new;
    }
    // ---- weights: their bf16 values on lanes g, the bf16 remainders on lanes G + g ----
    bf16x8 pw[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float pv = fast_exp2(s[v] - m_run);
      l_run += pv;
      pw[v >> 3][v & 7] = (__bf16)fmaf(-remainder, (float)(__bf16)pv, pv);
    }
    // ---- output: contraction index e of step ks on lane half `half` is tile row
    //      16 ks + 4 half + 8 (e / 4) + e % 4, the row accumulator register 8 ks + e holds ----
    if (LITERAL && literal) {
      // v_hat[t][j] = sum_i K[t][i] W[i][j] per 32-wide block of j: rows = tokens, so that the
      // accumulator of lane j holds its column in exactly the order the second product wants
      // for its A operand; fed as bf16 value + remainder like the weights.
#pragma unroll
      for (int jb = 0; jb < JB; ++jb) {
        const unsigned char* wt = dec_lds + jb * 2 * TL::kTileBytes + TL::kTileBytes;
        f32x16 vh;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          const u32x4 a = *reinterpret_cast<const u32x4*>(k_tile + l31 * TL::kStride + (2 * c + half) * 16);
          const u32x4 b = *reinterpret_cast<const u32x4*>(wt + l31 * TL::kStride + (2 * c + half) * 16);
          vh = mfma(a, b, c == 0 ? zero : vh);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          bf16x8 v_hi, v_lo;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float x = vh[8 * ks + e];
            const __bf16 hi = (__bf16)x;
            v_hi[e] = hi;
            v_lo[e] = (__bf16)(x - (float)hi);
          }
          o[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_hi, pw[ks], o[jb], 0, 0, 0);
          o[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_lo, pw[ks], o[jb], 0, 0, 0);
        }
      }
      return;
    }
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        typedef __attribute__((address_space(3))) s16x4 lds_quad;
        const uint32_t at = r_at + (uint32_t)(16 * ks * TL::kStride + jb * 64);
        const s16x4 a0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad*)(uintptr_t)at);
        const s16x4 a1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad*)(uintptr_t)(at + 8 * TL::kStride));
        const s16x8 a = __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
        o[jb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), pw[ks], o[jb], 0, 0, 0);
      }
    }
  };

  // Literal reconstruction: W^T of the head sits in the value-tile slots, which approximated rows
  // do not use (32 rows of W^T per slot, same row stride as a tile).
  if (LITERAL && literal) {
    const T* Wh = reinterpret_cast<const T*>(p.W) + (int64_t)h * p.w_sh;
    for (int idx = tid; idx < D * D / 8; idx += DT_) {
      const int i = idx / (D / 8), j0 = (idx % (D / 8)) * 8;
      union { uint4 raw; unsigned short el[8]; } w;
      w.raw = load_chunk(Wh + (size_t)i * D + j0);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int j = j0 + e;
        *reinterpret_cast<unsigned short*>(dec_lds + (j / 32) * 2 * TL::kTileBytes + TL::kTileBytes + (j % 32) * TL::kStride + i * 2) = w.el[e];
      }
    }
    __syncthreads();
  }

  // W for the weighted key sum: asked for before the rows, so that what waits for these has it
  const bool applies_w = APPLY && is_apx;
  if (applies_w) {
    const unsigned char* Wh = reinterpret_cast<const unsigned char*>(reinterpret_cast<const T*>(p.W) + (int64_t)h * p.w_sh);
    constexpr int kLoads = D * TL::kRowBytes / (kWave * 16) / DW;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int first = (wave * kLoads + i) * TL::kRowsPerLoad, row = first + ld_row, piece = ld_piece ^ TL::w_twist(row);
      load_to_lds16(lds_address(dec_lds) + TL::w_row(first), Wh + (size_t)row * TL::kRowBytes + piece * 16);
    }
  }
  int base = row_begin + wave * kTileRows;
  if (base < row_end) fetch(base);
  // The query rows have arrived from here on.  Without this the wait for them sits in the loop, in front of the first
  // product, and waits for the next tile's rows as well.
#pragma unroll
  for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(qf[c]));
  while (base < row_end) {
    wave_fence();                                    // last tile's reads are done before it is overwritten
    stage();
    const int next = base + kStepRows;
    if (next < row_end) fetch(next);     // in flight while this tile is consumed
    wave_fence();
    consume(base);
    base = next;
  }

  // ---- merge the waves ----
  const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
  if (APPLY) wave_fence();
  else __syncthreads();                              // every wave is done with its tiles: reuse the area
  // [DW][2 G][kRedStride]: weights' part, remainders' part; and [DW][2][G]
  constexpr int kRedWave = APPLY ? 2 * TL::kTileBytes / 4 : 2 * G * kRedStride, kMlWave = APPLY ? kRedWave : 2 * G;
  float* red = reinterpret_cast<float*>(dec_lds);
  float* ml = red + (APPLY ? 1 : DW) * 2 * G * kRedStride;
  if (l31 < 2 * G) {
#pragma unroll
    for (int jb = 0; jb < JB; ++jb)
#pragma unroll
      for (int v = 0; v < 16; v += 4) {
        const f32x4 x = {o[jb][v], o[jb][v + 1], o[jb][v + 2], o[jb][v + 3]};
        *reinterpret_cast<f32x4*>(red + wave * kRedWave + l31 * kRedStride + jb * 32 + acc_row(v, half)) = x;
      }
    if (half == 0 && l31 < G) {
      ml[wave * kMlWave + l31] = (l_tot > 0.f) ? m_run : -INFINITY;
      ml[wave * kMlWave + G + l31] = l_tot;
    }
  }
  if (applies_w) wait_loads<0>();
  __syncthreads();
  // a wave without rows has m = -inf and nothing but zeros: its share is 0 without a branch
  float* out = p.part + range.slot * PSZ;
  for (int i = tid * 4; i < G * D; i += DT_ * 4) {
    const int g = i / D, j = i % D;
    float mw[DW], m = -INFINITY, l = 0.f;
#pragma unroll
    for (int wv = 0; wv < DW; ++wv) { mw[wv] = ml[wv * kMlWave + g]; m = fmaxf(m, mw[wv]); }
    const float m_safe = m == -INFINITY ? 0.f : m;
    f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wv = 0; wv < DW; ++wv) {
      const float sc = fast_exp2(mw[wv] - m_safe);
      const f32x4 x = *reinterpret_cast<const f32x4*>(red + wv * kRedWave + g * kRedStride + j);
      const f32x4 y = *reinterpret_cast<const f32x4*>(red + wv * kRedWave + (G + g) * kRedStride + j);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = fmaf(x[e] + y[e], sc, a[e]);
      l = fmaf(ml[wv * kMlWave + G + g], sc, l);
    }
    if (applies_w) store_parts<TL::kStride>(dec_lds + TL::kParts + g * TL::kStride, j, a);
    else *reinterpret_cast<f32x4_u*>(out + 2 * G + i) = a;
    if (j == 0) {
      out[2 * g] = m;
      out[2 * g + 1] = l;
    }
  }
  if constexpr (APPLY) {
    if (!applies_w) return;
    __syncthreads();
    if (wave * 32 >= D) return;
    // W's columns by the transposing read, as in the merge
    typedef __attribute__((address_space(3))) s16x4 lds_quad;
    const int col = wave * 32 + ((lane >> 4) & 1) * 16 + 4 * (lane & 3);
    uint32_t w_at[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int row = 8 * k + 4 * half + (lane & 15) / 4;
      w_at[k] = lds_address(dec_lds) + TL::w_row(row) + (uint32_t)(((col / 8) ^ TL::w_twist(row)) * 16 + col % 8 * 2);
    }
    f32x16 acc;
#pragma unroll
    for (int c = 0; c < D / 16; ++c) {
      const s16x4 b0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad*)(uintptr_t)(w_at[0] + TL::w_row(16 * c) - TL::w_row(0)));
      const s16x4 b1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad*)(uintptr_t)(w_at[1] + TL::w_row(16 * c) - TL::w_row(0)));
      const u32x4 a = *reinterpret_cast<const u32x4*>(dec_lds + TL::kParts + min(l31, 23) * TL::kStride + (16 * c + 8 * half) * 2);
      acc = mfma(a, __builtin_bit_cast(u32x4, __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7)), c == 0 ? zero : acc);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int g = half * 4 + i;
      if (g < G) out[2 * G + g * D + wave * 32 + l31] = acc[i] + (acc[4 + i] + acc[8 + i]);
    }
  }
}
template <int D, int G, bool ROPE, bool LITERAL = false, bool PAGED = false, bool PLANNED = false, bool APPLY = false>
__global__ __launch_bounds__(DT_, 2) void decode_split_mfma_kernel(DecodeParams p, RopeParams rp) {
  for_split_rows<DW * kTileRows, PLANNED>(p, [&](const SplitRows& r, int tid) VEC_INLINE { attend_rows_mfma<D, G, ROPE, LITERAL, PAGED, APPLY>(p, rp, r, tid); });
}

// The partials of a (sequence, KV head): those of the retained segment from `first` on, then those of the approximated one, `gap`
// further on than the end of these
struct MergeSplits {
  int ret, apx, gap;
  size_t first;
  __device__ __forceinline__ size_t place(int split) const { return (size_t)(split + (split >= ret ? gap : 0)); }
};
template <bool PLANNED> __device__ __forceinline__ MergeSplits merge_splits(const DecodeParams& p, size_t bh) {
  if constexpr (PLANNED) {
    const int2 r = p.plan[2 * bh], a = p.plan[2 * bh + 1];
    return {r.y, a.y, r.y > 0 && a.y > 0 ? a.x - r.x - r.y : 0, (size_t)(r.y > 0 ? r.x : a.x)};
  } else {
    return {p.splits_ret, p.splits_apx, 0, bh * (p.splits_ret + p.splits_apx)};
  }
}

// LDS of the merge, bytes
template <typename T, int D, int G> struct CombineLds {
  static constexpr bool kMfma = sizeof(T) == 2;
  static constexpr int kQuads = G * D / 4;
  static constexpr int kSide = kQuads >= DT_ ? 1 : DT_ / kQuads;         // splits taken side by side
  static constexpr int kRounds = (kQuads + DT_ - 1) / DT_;
  static constexpr int kBlocks = (G + 7) / 8;                            // of eight query rows
  static constexpr int kStride = D * 2 + 16;                             // bytes of a row of W, and of z's parts
  static constexpr int kWeights = kMaxSplits * G * 4, kParts = kMfma ? kBlocks * 32 * kStride : DW * G * D * 4;      // not at the same time
  static constexpr int kSums = (kWeights > kParts ? kWeights : kParts);            // [2: retained, approximated][kSide][G * D]
  static constexpr int kW = kSums + 2 * kSide * G * D * 4;
  static constexpr int kInv = kW + (kMfma ? D * kStride : 0);
  static constexpr int kTotal = kInv + G * 4;
};

// Merge of the splits, one workgroup per (sequence, KV head): reference and sum of every query row, the weighted sums of the
// splits, z W, the division.  What bounds it is a chain: arguments, one trip to memory, weights, sums, z W.  Every load of the
// first splits is out before the first is waited for.  The splits' weights: a wave takes a query row, lane s its split s, so that the
// row's reference and sum are two reductions over the wave; a thread then takes four neighbouring elements of every kSide-th
// split with 16-byte loads, and the weights from LDS.
// bf16: z W runs on the matrix cores: z in three bf16 parts
// (its 24 bits, eight at a time, cut and not rounded: above bf16's largest number a rounded first part would be infinite, and
// the second minus infinity; of an infinite z the first part is all), eight query rows by three parts on the M side, W's
// columns by the transposing LDS read.  fp32: on the vector unit, a thread with 16 bytes of some rows of W.
// One sequence of 8192 tokens, 8 KV heads, 17 splits, W applied here (that launch's pieces apply it themselves now, which ends the chain
// at the sums): from the launch's start 0.9 us to the loads, 0.5 to the weights, 1.0 to the
// sums (W arrives), 0.3, and 0.8 for z W; with every thread looping over all splits' references the second and third took 2.2
// (a step 11.7 us, then 11.2).  In the split launch's last workgroup of a (sequence, KV head) instead of a launch of its
// own it is no faster: the acknowledgement of the written splits and the count of them take 1 us, as a launch does, and keep every
// workgroup on its CU that much longer (11.6 / 12.1, and with 16 sequences of 32768 tokens 70.6 / 72.8).
template <typename T, int D, int G, bool PLANNED = false>
__global__ __launch_bounds__(DT_) void decode_combine_kernel(DecodeParams p) {
  using L = CombineLds<T, D, G>;
  constexpr int kFlight = 8, PSZ = 2 * G + G * D;
  constexpr int E = Elem<T>::kPerChunk;    // elements of W per 16-byte load
  constexpr int CG = D / E;                // fp32: thread groups along a row of W
  constexpr int RG = DT_ / CG;             // thread groups along its rows (the contraction index)
  constexpr int WL = D * D / E / DT_;      // pieces of W per thread
  constexpr int RW = (G + DW - 1) / DW;    // query rows per wave
  static_assert(kMaxSplits <= kWave, "a lane per split");
  extern __shared__ __align__(16) unsigned char dec_lds[];
  unsigned char* lds = dec_lds;
  float* weight = reinterpret_cast<float*>(lds);                         // [G][splits]
  float* sums = reinterpret_cast<float*>(lds + L::kSums);
  float* inv = reinterpret_cast<float*>(lds + L::kInv);
  const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const size_t bh = (size_t)b * p.Hkv + h;
  const MergeSplits cut = merge_splits<PLANNED>(p, bh);
  const int n_splits = cut.ret + cut.apx, n_ret = p.only_values ? n_splits : cut.ret;
  const float* part = p.part + cut.first * PSZ;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5, l31 = lane & 31;
  const bool use_w = p.n_approx > 0 && !p.only_values;

  // the step's own token is now a row of the cache (the split launch has finished): one thread per
  // sequence makes it live, unless the block was full
  const bool advances = p.k_new && h == 0 && tid == 0;
  int live = 0, cap = p.cap_retain;
  if (advances) {
    live = p.len_retain[b];
    if (p.cap_retain_seq) cap = max(p.cap_retain_seq[b], 0);
  }
  // this thread's elements, and its first splits
  const int quad = tid % L::kQuads;
  int side = L::kSide > 1 ? tid / L::kQuads : 0;       // of a whole wave the same where it can be: then which split counts where is a scalar question
  if constexpr (L::kQuads % kWave == 0) side = __builtin_amdgcn_readfirstlane(side);
  const int sides = min(L::kSide, n_splits);
  const bool has_quad = side < sides;
  f32x4 x0[kFlight];
  auto load_splits = [&](int round, int s0, f32x4* x) VEC_INLINE {
    const int at = min(round * DT_ + quad, L::kQuads - 1) * 4;
#pragma unroll
    for (int u = 0; u < kFlight; ++u) {
      x[u] = *reinterpret_cast<const f32x4_u*>(part + cut.place(min(s0 + u * L::kSide, n_splits - 1)) * PSZ + 2 * G + at);
    }
  };
  uint4 wraw[WL];
  const T* Wh = reinterpret_cast<const T*>(p.W) + (int64_t)h * p.w_sh;
  const int cg = tid % CG, rg = tid / CG;
  auto load_w = [&]() VEC_INLINE {
    if (use_w) {
#pragma unroll
      for (int i = 0; i < WL; ++i) wraw[i] = load_chunk(L::kMfma ? Wh + (size_t)(i * DT_ + tid) * 8 : Wh + (size_t)(rg * WL + i) * D + cg * E);
    }
  };
  if (!L::kMfma) load_w();                       // the larger part of what is read
  float2 ml[RW];
#pragma unroll
  for (int i = 0; i < RW; ++i) ml[i] = *reinterpret_cast<const float2*>(part + cut.place(min(lane, n_splits - 1)) * PSZ + 2 * min(wave + i * DW, G - 1));
  load_splits(0, min(side, n_splits - 1), x0);
  if (L::kMfma) load_w();
#pragma unroll
  for (int i = 0; i < RW; ++i) {
    const int g = wave + i * DW;
    if (G % DW == 0 || g < G) {                  // uniform
      const float m = lane < n_splits ? ml[i].x : -INFINITY, top = wave_max_dpp(m);
      const float w = fast_exp2(m - (top == -INFINITY ? 0.f : top)), l = wave_sum_dpp(lane < n_splits ? ml[i].y * w : 0.f);
      if (lane < n_splits) weight[g * n_splits + lane] = w;
      if (lane == 0) inv[g] = l > 0.f ? 1.f / l : 0.f;
    }
  }
  if (advances) const_cast<int*>(p.len_retain)[b] = min(min(max(live, 0), cap) + 1, cap);
  __syncthreads();
#pragma unroll
  for (int round = 0; round < L::kRounds; ++round) {
    const int at = round * DT_ + quad, g = min(at * 4, G * D - 1) / D;
    f32x4 av = {0.f, 0.f, 0.f, 0.f}, az = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = side; s0 < n_splits; s0 += kFlight * L::kSide) {
      f32x4 x[kFlight];
      if (round == 0 && s0 == side) {
#pragma unroll
        for (int u = 0; u < kFlight; ++u) x[u] = x0[u];
      } else {
        load_splits(round, s0, x);
      }
#pragma unroll
      for (int u = 0; u < kFlight; ++u) {
        const int s = s0 + u * L::kSide;
        if (s < n_splits) {
          const float sc = weight[g * n_splits + s];
          if (s < n_ret) {                       // not by weights of 0: a share may be infinite
#pragma unroll
            for (int e = 0; e < 4; ++e) av[e] = fmaf(x[u][e], sc, av[e]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) az[e] = fmaf(x[u][e], sc, az[e]);
          }
        }
      }
    }
    if (has_quad && at < L::kQuads) {
      *reinterpret_cast<f32x4*>(sums + side * G * D + at * 4) = av;
      *reinterpret_cast<f32x4*>(sums + (L::kSide + side) * G * D + at * 4) = az;
    }
  }
  unsigned char* w_tile = lds + L::kW;
  if (L::kMfma && use_w) {
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int piece = i * DT_ + tid;
      *reinterpret_cast<uint4*>(w_tile + piece / (D / 8) * L::kStride + piece % (D / 8) * 16) = wraw[i];
    }
  }
  __syncthreads();
  // z, and (bf16) its parts: part q of query row g in row (g / 8) * 32 + q * 8 + g % 8
  for (int i = tid * 4; i < G * D; i += DT_ * 4) {
    const int g = i / D, j = i % D;
    f32x4 v = {0.f, 0.f, 0.f, 0.f}, z = {0.f, 0.f, 0.f, 0.f};
    for (int q = 0; q < sides; ++q) {
      v += *reinterpret_cast<const f32x4*>(sums + q * G * D + i);
      z += *reinterpret_cast<const f32x4*>(sums + (L::kSide + q) * G * D + i);
    }
    if (L::kSide > 1) *reinterpret_cast<f32x4*>(sums + i) = v;
    if (!L::kMfma) {
      if (L::kSide > 1) *reinterpret_cast<f32x4*>(sums + L::kSide * G * D + i) = z;
    } else if (use_w) {
      store_parts<L::kStride>(lds + ((g / 8) * 32 + g % 8) * L::kStride, j, z);
    }
  }
  __syncthreads();
  if constexpr (L::kMfma) {
    if (wave * 32 >= D) return;
    const int j = wave * 32 + l31;
    const uint32_t w_at = lds_address(w_tile) + (uint32_t)((4 * half + (lane & 15) / 4) * L::kStride + (wave * 32 + ((lane >> 4) & 1) * 16 + 4 * (lane & 3)) * 2);
#pragma unroll
    for (int blk = 0; blk < L::kBlocks; ++blk) {
      f32x16 acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
      if (use_w) {
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
          typedef __attribute__((address_space(3))) s16x4 lds_quad;
          const uint32_t at = w_at + (uint32_t)(16 * c * L::kStride);
          const s16x4 b0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad*)(uintptr_t)at);
          const s16x4 b1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad*)(uintptr_t)(at + 8 * L::kStride));
          const chunk_t a = *reinterpret_cast<const chunk_t*>(lds + (blk * 32 + min(l31, 23)) * L::kStride + (16 * c + 8 * half) * 2);
          mma_chunk<T>(acc, a, __builtin_bit_cast(chunk_t, __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7)));
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int g = blk * 8 + half * 4 + i;
        if (g < G) {
          const float r = (sums[g * D + j] + (acc[i] + (acc[4 + i] + acc[8 + i]))) * inv[g];
          const size_t at = ((size_t)b * p.Hq + (size_t)h * G + g) * D + j;
          if (p.out_f32) reinterpret_cast<float*>(p.out)[at] = r;
          else store_elem(reinterpret_cast<T*>(p.out) + at, r);
        }
      }
    }
  } else {
    // partial products over the thread's rows of W, summed over the row groups of a wave by lane exchange, over the waves
    // through LDS
    static_assert(CG <= kWave && D % RG == 0 && WL == D / RG, "a wave holds whole row groups");
    const float* z = sums + L::kSide * G * D;
    float (*zw)[G][D] = reinterpret_cast<float (*)[G][D]>(lds);
    float a[G][E];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < E; ++e) a[g][e] = 0.f;
    if (use_w) {
#pragma unroll
      for (int r = 0; r < WL; ++r) {
        float wf[E];
        Unpack16<T>::run(wraw[r], wf);
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float zg = z[g * D + rg * WL + r];
#pragma unroll
          for (int e = 0; e < E; ++e) a[g][e] = fmaf(zg, wf[e], a[g][e]);
        }
      }
    }
#pragma unroll
    for (int o = CG; o < kWave; o <<= 1)
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < E; ++e) a[g][e] += __shfl_xor(a[g][e], o, kWave);
    if (lane < CG) {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < E; ++e) zw[wave][g][cg * E + e] = a[g][e];
    }
    __syncthreads();
    T* out = reinterpret_cast<T*>(p.out) + ((size_t)b * p.Hq + (size_t)h * G) * D;
    for (int i = tid; i < G * D; i += DT_) {
      const int g = i / D, j = i % D;
      float sum = 0.f;
#pragma unroll
      for (int q = 0; q < DW; ++q) sum += zw[q][g][j];
      out[i] = (sums[i] + sum) * inv[g];
    }
  }
}

// The same for fp32 caches with few elements: two barriers less, every thread with its own weights.  A step, us, captured,
// this / decode_combine_kernel:
//   d = 64:  5 sequences of 1040 tokens, two query heads 7.3 / 8.0; 27 of 2052, four 29.1 / 29.5; one of 747, eight 12.3 / 12.6
//   d = 128: 23 of 1386, one 9.4 / 10.1; 3 of 673, two 10.6 / 10.5; one of 1153, four 14.3 / 12.9; 4 of 3461, four 19.9 / 16.4;
//            one of 2440, eight 28.1 / 24.4
template <int D, int G>
__global__ __launch_bounds__(256) void decode_combine_few_kernel(DecodeParams p) {
  using T = float;
  constexpr int PSZ = 2 * G + G * D;
  constexpr int E = Elem<T>::kPerChunk;    // elements of W per 16-byte load
  constexpr int CG = D / E;                // thread groups along a row of W
  constexpr int RG = 256 / CG;             // thread groups along its rows (the contraction index)
  constexpr int RP = D / RG;               // rows of W per thread
  constexpr int kWavesC = 256 / kWave;
  static_assert(CG <= kWave && D % RG == 0, "a wave holds whole row groups");
  __shared__ float z_lds[G][D];
  __shared__ float v_lds[G][D];
  __shared__ float zw_lds[kWavesC][G][D];
  __shared__ float linv_lds[G];
  const int h = blockIdx.x, b = blockIdx.y;
  const size_t bh = (size_t)b * p.Hkv + h;
  const int n_splits = p.splits_ret + p.splits_apx;
  const float* part = p.part + bh * n_splits * PSZ;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

  // this thread's block of W (rows rg*RP.., 16 bytes of each) is requested first: it depends on
  // nothing and arrives while the splits are merged
  const int cg = threadIdx.x % CG, rg = threadIdx.x / CG;
  const T* Wh = reinterpret_cast<const T*>(p.W) + (int64_t)h * p.w_sh;
  uint4 wraw[RP];
  const bool use_w = p.n_approx > 0;
  // the step's own token is now a row of the cache (the split launch has finished): one thread per
  // sequence makes it live, unless the block was full
  if (p.k_new && h == 0 && threadIdx.x == 0) {
    const int cap = p.cap_retain_seq ? max(p.cap_retain_seq[b], 0) : p.cap_retain;
    int* len = const_cast<int*>(p.len_retain) + b;
    *len = min(min(max(*len, 0), cap) + 1, cap);
  }
  if (use_w) {
#pragma unroll
    for (int r = 0; r < RP; ++r) wraw[r] = load_chunk(Wh + (size_t)(rg * RP + r) * D + cg * E);
  }

  // A thread owns G*D/256 output elements and, for each, reads every split's (m, l, partial) itself (the (m, l)
  // reads of a query row are shared by the lanes that work on that row).  The reads of up to four elements and of 8 or
  // 16 splits go out together and are folded into running maxima.  One element and eight splits at a time, a step of one sequence of
  // 4096 tokens, d = 128, took 18.4 us against 16.8 with four query heads, 32.0 against 27.6 with eight.
  constexpr int NE = (G * D + 255) / 256, EB = NE < 4 ? NE : 4;
  auto fold_splits = [&](auto fold_tag) __attribute__((always_inline)) {
    constexpr int kFold = decltype(fold_tag)::value;
    for (int e0 = 0; e0 < NE; e0 += EB) {
      float M[EB], L[EB], av[EB], az[EB];
#pragma unroll
      for (int e = 0; e < EB; ++e) { M[e] = -INFINITY; L[e] = av[e] = az[e] = 0.f; }
      for (int s0 = 0; s0 < n_splits; s0 += kFold) {
        float ms[EB][kFold], ls[EB][kFold], xs[EB][kFold];
#pragma unroll
        for (int u = 0; u < kFold; ++u) {
          const float* at = part + (size_t)min(s0 + u, n_splits - 1) * PSZ;
#pragma unroll
          for (int e = 0; e < EB; ++e) {
            const int i = min((int)threadIdx.x + (e0 + e) * 256, G * D - 1), g = i / D;
            ms[e][u] = at[2 * g];
            ls[e][u] = at[2 * g + 1];
            xs[e][u] = at[2 * G + i];
          }
        }
#pragma unroll
        for (int e = 0; e < EB; ++e) {
          float mx = M[e];
#pragma unroll
          for (int u = 0; u < kFold; ++u)
            if (s0 + u < n_splits) mx = fmaxf(mx, ms[e][u]);
          const float keep = (M[e] == -INFINITY) ? 0.f : fast_exp2(M[e] - mx);     // mx = -inf only if M is
          L[e] *= keep; av[e] *= keep; az[e] *= keep;
#pragma unroll
          for (int u = 0; u < kFold; ++u) {
            if (s0 + u < n_splits && ms[e][u] != -INFINITY) {
              const float sc = fast_exp2(ms[e][u] - mx);
              L[e] = fmaf(ls[e][u], sc, L[e]);
              if (s0 + u < p.splits_ret) av[e] = fmaf(xs[e][u], sc, av[e]);
              else az[e] = fmaf(xs[e][u], sc, az[e]);
            }
          }
          M[e] = mx;
        }
      }
#pragma unroll
      for (int e = 0; e < EB; ++e) {
        const int i = (int)threadIdx.x + (e0 + e) * 256;
        if (e0 + e < NE && i < G * D) {
          (&v_lds[0][0])[i] = av[e];
          (&z_lds[0][0])[i] = az[e];
          if (i % D == 0) linv_lds[i / D] = (L[e] > 0.f) ? 1.f / L[e] : 0.f;
        }
      }
    }
  };
  if (n_splits > 8 && EB <= 2) fold_splits(std::integral_constant<int, EB <= 2 ? 16 : 8>{});
  else fold_splits(std::integral_constant<int, 8>{});
  __syncthreads();
  // out[g][j] = (sum_ret p v  +  z[g][:] . W[:, j]) / l : partial products over the thread's rows
  // of W, summed over the row groups of a wave by lane exchange, over the waves through LDS
  {
    float a[G][E];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int e = 0; e < E; ++e) a[g][e] = 0.f;
    if (use_w) {
#pragma unroll
      for (int r = 0; r < RP; ++r) {
        float wf[E];
        Unpack16<T>::run(wraw[r], wf);
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const float zg = z_lds[g][rg * RP + r];
#pragma unroll
          for (int e = 0; e < E; ++e) a[g][e] = fmaf(zg, wf[e], a[g][e]);
        }
      }
    }
#pragma unroll
    for (int o = CG; o < kWave; o <<= 1)
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < E; ++e) a[g][e] += __shfl_xor(a[g][e], o, kWave);
    if (lane < CG) {
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int e = 0; e < E; ++e) zw_lds[wave][g][cg * E + e] = a[g][e];
    }
  }
  __syncthreads();
  T* out = reinterpret_cast<T*>(p.out) + ((size_t)b * p.Hq + (size_t)h * G) * D;
  for (int i = threadIdx.x; i < G * D; i += 256) {
    const int g = i / D, j = i % D;
    float zw = 0.f;
#pragma unroll
    for (int q = 0; q < kWavesC; ++q) zw += zw_lds[q][g][j];
    out[i] = (v_lds[g][j] + zw) * linv_lds[g];
  }
}

template <typename T, int D, int G> constexpr bool kFewElements = sizeof(T) == 4 && (D == 64 ? G <= 8 : G <= 2);

// Workgroups of a split kernel that fit a CU, asked for once per kernel.
template <auto Kernel> int workgroups_per_cu(int lds) {
  static const int n = [&] {
    int fit = 0;
    if (set_max_lds(reinterpret_cast<const void*>(Kernel), lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit, reinterpret_cast<const void*>(Kernel), DT_, lds) != hipSuccess) (void)hipGetLastError();
    return fit > 0 ? fit : 1;
  }();
  return n;
}

// Applying: the kernel for plain rows where a small launch applies W (APPLY), or Kernel
template <auto Kernel, typename T, int D, int G, auto Applying = Kernel>
int launch_split(const vector_cache& c, DecodeParams& p, int lds, hipStream_t stream, const RopeParams* rope) {
  const ApproxRows kind = rope ? ApproxRows::kTurned : p.literal ? ApproxRows::kRebuilt : ApproxRows::kPlain;
  const SplitCosts costs = split_costs(Elem<T>::kDtype == VECTOR_BF16, D, G, kind, workgroups_per_cu<Kernel>(lds));
  static_assert(Elem<T>::kDtype == VECTOR_BF16 ? DW * kTileRows == 128 : DW * kWave * 4 * kUnroll == 4096, "the rows of a step that split_costs states");
  // paged: a range's block ids fit a register across the wave, see tile_in_block
  const int least_ret = c.ret_block_table ? (int)(((int64_t)c.cap_retain + (int64_t)(kWave - 1) * c.ret_block_rows - 1) / ((int64_t)(kWave - 1) * c.ret_block_rows)) : 1;
  p.by_kind = kind == ApproxRows::kPlain && costs.one_round &&
              pick_one_round(costs, c.batch, c.n_kv_heads, c.cap_retain, c.n_approx, least_ret, p.splits_ret, p.splits_apx);
  if (!p.by_kind) pick_splits(costs, c.batch, c.n_kv_heads, c.cap_retain, c.n_approx, p.splits_ret, p.splits_apx);
  // As long as a CU has one workgroup: the pieces of approximated rows wait for W beside their rows, and the merge has less to wait
  // for.  With two, W's share of what they wait for is longer than what the merge loses.  A step without / with, us: one sequence of
  // 8192 tokens 10.3 / 9.8, of 30000 14.7 / 14.1, two of 32768 16.0 / 15.1, three of 8192 13.6 / 13.1 (192 workgroups);
  // four 14.6 / 15.2 (352), 16 30.9 / 31.7, ten of 32768 45.2 / 46.2.  A kernel of its own: as a branch of the other one its 1.5 KB of
  // code had to come into the instruction cache of every launch (one sequence of 8192 tokens 9.8 / 9.7).
  const bool apply_w = Applying != Kernel && c.n_approx > 0 && (int64_t)c.batch * c.n_kv_heads * (p.splits_ret + p.splits_apx) <= 256;
  const unsigned splits = p.splits_ret + p.splits_apx, heads = c.n_kv_heads, batch = c.batch;
  const dim3 grid = p.by_kind ? dim3(heads, batch, splits) : dim3(splits, heads, batch);
  if constexpr (Applying != Kernel) {
    if (apply_w) {
      constexpr int more_lds = MfmaDecodeTile<D>::kLdsBytes;
      VEC_HIP(set_max_lds(reinterpret_cast<const void*>(Applying), more_lds));
      VEC_LAUNCH(K_DECODE_SPLIT, Applying, grid, dim3(DT_), more_lds, stream, p, RopeParams{});
      p.only_values = 1;
      return VECTOR_OK;
    }
  }
  VEC_HIP(set_max_lds(reinterpret_cast<const void*>(Kernel), lds));
  VEC_LAUNCH(K_DECODE_SPLIT, Kernel, grid, dim3(DT_), lds, stream, p, rope ? *rope : RopeParams{});
  return VECTOR_OK;
}

// Sequences of different lengths, and their merge
template <auto Kernel, typename T, int D, int G>
int launch_planned(const vector_cache& c, DecodeParams& p, hipStream_t stream, const RopeParams* rope) {
  constexpr int lds = MfmaDecodeTile<D>::kTiles, merge_lds = CombineLds<T, D, G>::kTotal;
  constexpr auto merge = decode_combine_kernel<T, D, G, true>;
  VEC_HIP(set_max_lds(reinterpret_cast<const void*>(Kernel), lds));
  VEC_HIP(set_max_lds(reinterpret_cast<const void*>(merge), merge_lds));
  const int pairs = c.batch * c.n_kv_heads;
  p.plan_apx = rope ? kPlanTurned : 1.f;
  p.plan = reinterpret_cast<int2*>(p.part + (size_t)pairs * kMaxSplits * (2 * G + G * D));      // behind the partials, half of the workspace
  const int per_cu = workgroups_per_cu<Kernel>(lds), wgs = plan_workgroups(per_cu, pairs);
  p.plan_most_retained = plan_most_retained(per_cu, wgs);
  VEC_LAUNCH(K_DECODE_SPLIT, Kernel, dim3(wgs), dim3(DT_), lds, stream, p, rope ? *rope : RopeParams{});
  VEC_LAUNCH(K_DECODE_COMBINE, merge, dim3(c.n_kv_heads, c.batch), dim3(DT_), merge_lds, stream, p);
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

template <typename T, int D, int G, bool PAGED>
int run_decode_layout(const vector_cache& c, DecodeParams& p, hipStream_t stream, const RopeParams* rope) {
  int rc;
  if constexpr (!PAGED && Elem<T>::kDtype == VECTOR_BF16) {
    if (c.cap_retain_seq && !p.literal) {
      constexpr int lds = MfmaDecodeTile<D>::kTiles;
      if constexpr (D == 128) {
        constexpr auto turned = decode_split_mfma_kernel<D, G, true, false, false, true>;
        if (rope && worth_a_plan(D, true, workgroups_per_cu<turned>(lds), c.batch, c.n_kv_heads, c.cap_retain, c.n_approx))
          return launch_planned<turned, T, D, G>(c, p, stream, rope);
      }
      constexpr auto plain = decode_split_mfma_kernel<D, G, false, false, false, true>;
      if (!rope && worth_a_plan(D, false, workgroups_per_cu<plain>(lds), c.batch, c.n_kv_heads, c.cap_retain, c.n_approx))
        return launch_planned<plain, T, D, G>(c, p, stream, rope);
    }
  }
  if constexpr (Elem<T>::kDtype == VECTOR_BF16) {
    constexpr int lds = MfmaDecodeTile<D>::kTiles;
    if (rope) rc = launch_split<decode_split_mfma_kernel<D, G, true, false, PAGED>, T, D, G>(c, p, lds, stream, rope);
    else if (p.literal) rc = launch_split<decode_split_mfma_kernel<D, G, false, true, PAGED>, T, D, G>(c, p, lds, stream, rope);
    else rc = launch_split<decode_split_mfma_kernel<D, G, false, false, PAGED>, T, D, G, decode_split_mfma_kernel<D, G, false, false, PAGED, false, (G <= kMostApplying)>>(
        c, p, lds, stream, rope);
  } else {
    if (rope) rc = launch_split<decode_split_kernel<T, D, G, PAGED, true>, T, D, G>(c, p, 0, stream, rope);
    else rc = launch_split<decode_split_kernel<T, D, G, PAGED, false>, T, D, G>(c, p, 0, stream, rope);
  }
  if (rc != VECTOR_OK) return rc;
  const dim3 merge_grid(c.n_kv_heads, c.batch);
  if constexpr (kFewElements<T, D, G>) {
    VEC_LAUNCH(K_DECODE_COMBINE, (decode_combine_few_kernel<D, G>), merge_grid, dim3(DT_), 0, stream, p);
  } else {
    constexpr int lds = CombineLds<T, D, G>::kTotal;
    VEC_HIP(set_max_lds(reinterpret_cast<const void*>(decode_combine_kernel<T, D, G>), lds));
    VEC_LAUNCH(K_DECODE_COMBINE, (decode_combine_kernel<T, D, G>), merge_grid, dim3(DT_), lds, stream, p);
  }
  VEC_HIP(hipGetLastError());
  return VECTOR_OK;
}

template <typename T, int D, int G>
int run_decode(const vector_cache& c, DecodeParams& p, hipStream_t stream, const RopeParams* rope) {
  return p.block_table ? run_decode_layout<T, D, G, true>(c, p, stream, rope) : run_decode_layout<T, D, G, false>(c, p, stream, rope);
}

template <typename T, int D>
int run_decode_g(const vector_cache& c, DecodeParams& p, hipStream_t stream, const RopeParams* rope) {
  switch (c.n_q_heads / c.n_kv_heads) {
    case 1: return run_decode<T, D, 1>(c, p, stream, rope);
    case 2: return run_decode<T, D, 2>(c, p, stream, rope);
    case 3: return run_decode<T, D, 3>(c, p, stream, rope);
    case 4: return run_decode<T, D, 4>(c, p, stream, rope);
    case 5: return run_decode<T, D, 5>(c, p, stream, rope);
    case 6: return run_decode<T, D, 6>(c, p, stream, rope);
    case 7: return run_decode<T, D, 7>(c, p, stream, rope);
    case 8: return run_decode<T, D, 8>(c, p, stream, rope);
    case 10: return run_decode<T, D, 10>(c, p, stream, rope);
    case 12: return run_decode<T, D, 12>(c, p, stream, rope);
    case 16: return run_decode<T, D, 16>(c, p, stream, rope);
    default: return VECTOR_ERR_SHAPE;
  }
}

}  // namespace

size_t decode_workspace_bytes(int batch, int n_q_heads, int n_kv_heads, int head_dim, int cap_retain, int n_approx) {
  // sized for the largest split count so that the bound holds for any live length (twice what a launch writes; a planned
  // one keeps its plan in the other half)
  (void)cap_retain; (void)n_approx;
  const int G = n_q_heads / n_kv_heads;
  return align_up((size_t)batch * n_kv_heads * 2 * kMaxSplits * (2 * G + G * head_dim) * sizeof(float), 256);
}

int launch_decode_attn(const vector_cache& c, const void* q, float scale, void* out, int flags, void* ws,
                       hipStream_t stream, const RopeParams* rope, const void* k_new, const void* v_new) {
  DecodeParams p;
  p.literal = (flags & VECTOR_DECODE_LITERAL) ? 1 : 0;
  p.only_values = p.literal;
  p.out_f32 = (flags & VECTOR_DECODE_OUT_F32) ? 1 : 0;
  if (p.literal && (rope || c.dtype != VECTOR_BF16)) return VECTOR_ERR_DTYPE;
  p.q = q; p.k_ret = c.k_ret; p.v_ret = c.v_ret; p.k_apx = c.k_apx; p.W = c.W; p.len_retain = c.len_retain;
  p.k_new = k_new; p.v_new = v_new;
  p.block_table = c.ret_block_table; p.block_shift = 0; p.blocks_per_seq = c.ret_blocks_per_seq;
  while (c.ret_block_table && (1 << p.block_shift) < c.ret_block_rows) ++p.block_shift;
  p.cap_retain_seq = c.cap_retain_seq; p.n_approx_seq = c.n_approx_seq;
  p.ret_row_start = c.ret_row_start; p.apx_row_start = c.apx_row_start;
  p.out = out; p.part = reinterpret_cast<float*>(ws);
  p.B = c.batch; p.Hq = c.n_q_heads; p.Hkv = c.n_kv_heads; p.cap_retain = c.cap_retain; p.n_approx = c.n_approx;
  p.w_sh = c.w_shared ? 0 : (int64_t)c.head_dim * c.head_dim;
  p.c2 = scale * kLog2e;
  p.plan = nullptr;
  p.plan_apx = 0.f;
  p.plan_most_retained = 0;
  p.by_kind = 0;
  if (c.dtype == VECTOR_BF16) {
    if (c.head_dim == 128) return run_decode_g<bf16_t, 128>(c, p, stream, rope);
    if (c.head_dim == 64) return run_decode_g<bf16_t, 64>(c, p, stream, rope);
  } else if (c.dtype == VECTOR_F32) {
    if (c.head_dim == 128) return run_decode_g<float, 128>(c, p, stream, rope);
    if (c.head_dim == 64) return run_decode_g<float, 64>(c, p, stream, rope);
  } else {
    return VECTOR_ERR_DTYPE;
  }
  return VECTOR_ERR_SHAPE;
}

}  // namespace vec
