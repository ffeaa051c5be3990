// Importance score (observation-window attention mass, pooled) and
// reconstruction residual ||v - k W||^2 for the VECTOR compression pass
// (Section 3.2, Steps 1 and 2).
//
// Data flow per KV head h (R = G*w query rows share the head's keys):
//   pass 1  score_stats   : S = Q_h K_h^T (MFMA), per-row sum-exp against a reference
//                           over a chunk of tokens -> partial (m, l) per (row, chunk)
//   pass 2  mass_residual : prologue merges the chunk partials into one bias per row,
//                           bias_r = log2-domain reference + log2(sum-exp); then S again,
//                           p = exp2(S*c - bias_r), column mean -> mass; fused on the
//                           same keys: v_hat^T = W^T K^T (MFMA),
//                           eps = sum_j (v - v_hat)^2
//   pool                  : average or maximum pooling of mass over prefix columns, +inf on the
//                           window columns (in the routing's launches: route_head.hip, or
//                           route_bucket_kernel in route_compact.hip for long heads)
//
// The kernels are in score_stream.hpp; this file decides how the tokens are split over workgroups and
// chunks, and which kernel runs.  Both passes put all chunks of a KV head on one XCD.
#include <algorithm>

#include "plan.hpp"
#include "score_stream.hpp"

namespace vec {

namespace {

// How many tokens a workgroup takes (a multiple of `tile`), so that `count` sequences of n[b] tokens, each
// with `heads` heads, make at most one workgroup per CU: their LDS lets one run on a CU at a time, and a
// second, nearly empty round would cost as much as the first.  With more than 128 heads, of which one round could
// take one workgroup each and leave up to half the chip idle, about four rounds of smaller ones instead.
// Stacked prompts of 8 heads, a compression pass in us, four rounds against one:
//     heads     1024       2048       4100       8192      16000 tokens
//      136    76 /  58   97 /  94  159 / 152  269 / 285  481 /  529
//      192    72 /  60  118 /  97  203 / 175  347 / 330  638 /  636
//      256    91 /  66  152 / 118  247 / 210  446 / 402  798 /  790
//      384   107 / 110  205 / 214  349 / 363  630 / 692 1201 / 1322
// The line holds where the heads do not fill whole rounds and the prompts are long; for short ones, and for a
// multiple of 256 heads, one round would be better.  Up to 128 heads it is better throughout (64 heads, four rounds
// against one: 56 / 30 at 1024 tokens, 236 / 210 at 16000).
int tokens_per_workgroup(const int* n, int count, int64_t heads, int tile) {
  const int64_t target = heads * count > 128 ? 1024 : 256;
  auto workgroups = [&](int64_t tiles) {
    int64_t total = 0;
    for (int b = 0; b < count; ++b) total += heads * ((n[b] + tiles * tile - 1) / (tiles * tile));
    return total;
  };
  int64_t most = 1;
  for (int b = 0; b < count; ++b) most = std::max<int64_t>(most, (n[b] + tile - 1) / tile);
  return (int)(smallest_step(most, target, workgroups) * tile);
}
constexpr int kMaxChunks = 256;                 // per head; reached by a single head

int units_of(int rows) { return rows <= 128 ? 4 : rows <= 256 ? 8 : 16; }

int stream_tile_tokens(int dtype, int head_dim) { return kStreamTileBytes / (head_dim * (dtype == VECTOR_BF16 ? 2 : 4)); }

}  // namespace

// Partials for the longest row block of any group, and the most chunks that any plan gives a head: kMaxChunks, of a tile
// of tokens at least.  A plan for several heads has fewer (256 over the number of heads), but s may be sequences
// stacked, each with the chunks it would have alone, and how many heads those have the shape does not say.
static size_t partial_bytes(const vector_shape& s) {
  const int64_t rows = (int64_t)(s.n_q_heads / s.n_kv_heads) * s.window;
  const int64_t tile = stream_tile_tokens(s.dtype, s.head_dim);
  const int64_t chunks = std::min<int64_t>((s.seq_len + tile - 1) / tile, kMaxChunks);
  return align_up((size_t)s.n_kv_heads * chunks * units_of((int)std::min<int64_t>(rows, 512)) * 32 * sizeof(float2), 256);
}

size_t score_workspace_bytes(const vector_shape& s) {
  return partial_bytes(s) + align_up((size_t)s.n_kv_heads * s.seq_len * sizeof(float), 256);
}

float* score_mass(const vector_shape& s, void* ws) {
  return reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(ws) + partial_bytes(s));
}

// One pair of passes over the keys for the query rows [q_row0, q_row0 + rows of `g`) of every KV
// head (g: the shape with the group's query-head count).  accumulate: the column mass is added to
// what earlier groups left.  The residual rides along when eps is given.  prepare_passes fills in
// the parameters, launch_passes enqueues the kernels (ragged: one launch for several sequences'
// parameter blocks, see PassParams::seq_table).
// plan_heads / plan_wg: chunks are laid out for one sequence's own heads, whatever else is in the launch, so that
// a sequence gets the same partials (and with them the same bits) as alone; a workgroup then takes as many
// chunks as make up plan_wg tokens.
template <typename T, int D>
static int prepare_passes(const SeqStack* stack, const vector_shape& s, const vector_shape& g, int q_row0, bool accumulate, const void* q,
                          const void* k, const void* v, const void* W, bool do_mass, float* eps, void* ws, const RopeParams* rope,
                          const QueryLse* lse, float4* range, int plan_wg, PassLaunch& L) {
  constexpr int kTile = Stream<T, D>::kTokens;
  L.do_mass = do_mass;
  L.do_res = eps != nullptr;
  PassParams& p = L.pp;
  p = PassParams{};
  const int rows = (g.n_q_heads / g.n_kv_heads) * g.window, rows_all = (s.n_q_heads / s.n_kv_heads) * s.window;
  if (do_mass && rows > kMaxUnits<T, D> * 32) return VECTOR_ERR_SHAPE;
  L.units = units_of(rows);
  p.n = s.seq_len; p.w = s.window; p.R = rows; p.R_pad = L.units * 32;
  p.n_prefix = s.seq_len - s.window;
  p.q_head_rows = rows_all; p.q_row0 = q_row0; p.accumulate = accumulate ? 1 : 0;
  p.c2 = kLog2e / sqrtf((float)D);
  p.inv_R = 1.0f / (float)rows_all;
  p.k_st = s.k_stride_tok ? s.k_stride_tok : D;
  p.k_sh = s.k_stride_head ? s.k_stride_head : (int64_t)s.seq_len * p.k_st;
  p.v_st = s.v_stride_tok ? s.v_stride_tok : D;
  p.v_sh = s.v_stride_head ? s.v_stride_head : (int64_t)s.seq_len * p.v_st;
  p.w_sh = s.w_shared ? 0 : (s.w_stride_head ? s.w_stride_head : (int64_t)D * D);
  if (stack) {                      // the strides inside a sequence are the shape's, as for one sequence
    p.hps = stack->heads_per_seq; p.k_sb = stack->k_stride_seq; p.v_sb = stack->v_stride_seq;
  }
  p.q = q; p.k = k; p.v = v; p.W = W; p.eps = eps; p.repeat = 1;
  p.range = do_mass ? range : nullptr;
  if (lse && do_mass) { p.lse = lse->lse; p.lse_sh = lse->stride_head ? lse->stride_head : s.window; }
  p.log_ref = -log2f((float)(p.n_prefix > 0 ? p.n_prefix : 1));
  p.part = reinterpret_cast<float2*>(ws);
  p.mass = ws ? score_mass(s, ws) : nullptr;

  p.tokens_per_wg = plan_wg ? plan_wg : tokens_per_workgroup(&s.seq_len, 1, s.n_kv_heads, kTile);
  p.tpc1 = tokens_per_workgroup(&s.seq_len, 1, stack ? stack->heads_per_seq : s.n_kv_heads, kTile);
  p.n_chunks = (s.seq_len + p.tpc1 - 1) / p.tpc1;
  p.chunks_per_wg = std::max(1, (p.tokens_per_wg + p.tpc1 - 1) / p.tpc1);
  if (p.n_chunks > kMaxChunks) return VECTOR_ERR_SHAPE;
  L.rp = RopeParams{};
  L.use_rope = rope != nullptr && L.do_res;                // the scores use the keys as cached
  if (L.use_rope) L.rp = *rope;
  L.grid1 = dim3((p.n_chunks + p.chunks_per_wg - 1) / p.chunks_per_wg, s.n_kv_heads);
  L.grid2 = dim3((s.seq_len + p.tokens_per_wg - 1) / p.tokens_per_wg, s.n_kv_heads);
  p.wgs1 = (int)L.grid1.x;
  p.range_stride = (int)L.grid2.x;
  return VECTOR_OK;
}

template <typename T, int D>
static int run_passes(const SeqStack* stack, const vector_shape& s, const vector_shape& g, int q_row0, bool accumulate, const void* q,
                      const void* k, const void* v, const void* W, bool do_mass, float* eps, void* ws, hipStream_t stream,
                      const RopeParams* rope, const QueryLse* lse, float4* range, int* n_range_out, float** mass_out, int* n_prefix_out) {
  PassLaunch L;
  const int rc = prepare_passes<T, D>(stack, s, g, q_row0, accumulate, q, k, v, W, do_mass, eps, ws, rope, lse, range, 0, L);
  if (rc != VECTOR_OK) return rc;
  if (mass_out) *mass_out = L.pp.mass;
  if (n_prefix_out) *n_prefix_out = L.pp.n_prefix;
  if (n_range_out) *n_range_out = (int)L.grid2.x;
  PassArgs<false> args = {{L.pp}};
  return launch_passes<T, D, false>(args, L, stream);
}

// Query heads per pair of passes: all G of a KV head when their G * w rows fit the kernels, else the largest
// count that does (0: one head's window is longer than the interface allows: the lengths that vector_score states.  The
// kernels would take any of kMaxUnits * 32 rows; fp32 at d = 128 has no more than its 256.)
template <typename T, int D>
static int heads_per_group(const vector_shape& s) {
  constexpr int kMaxWindow = sizeof(T) == 4 ? (D == 128 ? 256 : 288) : (D == 128 ? 288 : 384);
  if (s.window > kMaxWindow) return 0;
  return std::min(s.n_q_heads / s.n_kv_heads, kMaxUnits<T, D> * 32 / s.window);
}

// Several sequences of different lengths, each with all its query heads in one group and its own
// score workspace: one pair of passes for all of them, then one pooling launch.
template <typename T, int D>
static int run_score_residual_ragged(const vector_shape& s, const RaggedSeq* seqs, int count, const void* W, void* tables,
                                     hipStream_t stream, const RopeParams* rope, bool leave_mass) {
  if (count < 1 || count > kMaxRaggedSeqs) return VECTOR_ERR_ARG;
  PassParams host[kMaxRaggedSeqs];
  PassLaunch first;
  unsigned g1 = 0, g2 = 0;                      // workgroups of the launches
  uint16_t first1[kMaxRaggedSeqs], first2[kMaxRaggedSeqs];
  std::fill(first1, first1 + kMaxRaggedSeqs, 0xffff);
  std::fill(first2, first2 + kMaxRaggedSeqs, 0xffff);
  int lens[kMaxRaggedSeqs];
  for (int b = 0; b < count; ++b) lens[b] = seqs[b].shape.seq_len;
  const int plan_wg = tokens_per_workgroup(lens, count, s.n_kv_heads, Stream<T, D>::kTokens);
  for (int b = 0; b < count; ++b) {
    vector_shape t = seqs[b].shape;
    if (heads_per_group<T, D>(t) != t.n_q_heads / t.n_kv_heads) return VECTOR_ERR_SHAPE;
    PassLaunch L;
    float4* range = leave_mass ? nullptr : reinterpret_cast<float4*>(route_mass_range(seqs[b].route_ws, t.n_kv_heads));
    const QueryLse ql = {seqs[b].lse, seqs[b].lse_stride_head};
    const int rc = prepare_passes<T, D>(nullptr, t, t, 0, false, seqs[b].q, seqs[b].k, seqs[b].v, W, true, seqs[b].eps, seqs[b].score_ws,
                                        rope, seqs[b].lse ? &ql : nullptr, range, plan_wg, L);
    if (rc != VECTOR_OK) return rc;
    L.pp.pos_base = seqs[b].pos_base;
    host[b] = L.pp;
    if (b == 0) first = L;
    first1[b] = (uint16_t)g1;
    first2[b] = (uint16_t)g2;
    g1 += L.grid1.x * s.n_kv_heads;
    g2 += L.grid2.x * s.n_kv_heads;
    if (std::max(g1, g2) > 0xffff) return VECTOR_ERR_SHAPE;      // cannot be: about 1024 are planned, or one per head, and a part has fewer heads
  }
  unsigned char* t8 = reinterpret_cast<unsigned char*>(tables);
  PassArgs<true> args;
  int rc = ragged_args(host, count, s.n_kv_heads, t8, stream, args);
  if (rc != VECTOR_OK) return rc;
  first.grid1 = dim3(g1);
  first.grid2 = dim3(g2);
  std::copy(first1, first1 + kMaxRaggedSeqs, first.first1);
  std::copy(first2, first2 + kMaxRaggedSeqs, first.first2);
  if ((rc = launch_passes<T, D, true>(args, first, stream)) != VECTOR_OK) return rc;
  if (leave_mass) return VECTOR_OK;
  // pooling + score-key buckets of every sequence
  PoolSeq pool[kMaxRaggedSeqs];
  for (int b = 0; b < count; ++b) {
    pool[b].mass = host[b].mass; pool[b].score = seqs[b].score; pool[b].eps = seqs[b].eps; pool[b].seq_len = seqs[b].shape.seq_len;
    pool[b].n_prefix = host[b].n_prefix; pool[b].route_ws = seqs[b].route_ws; pool[b].n_range = host[b].range_stride;
  }
  return launch_pool_scores_ragged(pool, count, s.n_kv_heads, s.pool_kernel, s.pool_mode, t8 + align_up(sizeof(PassParams) * count, 256), stream);
}

template <typename T, int D>
static int run_score_residual(const SeqStack* stack, const vector_shape& s, const void* q, const void* k, const void* v, const void* W,
                              float* score, float* eps, void* ws, hipStream_t stream, const RopeParams* rope,
                              void* route_ws, const QueryLse* lse, bool leave_mass) {
  const bool do_mass = score != nullptr;
  if (!do_mass) return run_passes<T, D>(stack, s, s, 0, false, q, k, v, W, false, eps, ws, stream, rope, nullptr, nullptr, nullptr, nullptr, nullptr);
  // The query heads of a KV head go through the two passes a group at a time; usually one group.
  // The first group's second pass carries the residual.
  const int G = s.n_q_heads / s.n_kv_heads;
  const int gh = heads_per_group<T, D>(s);
  if (gh == 0) return VECTOR_ERR_SHAPE;
  float* mass = nullptr;
  int n_prefix = 0, n_range = 0;
  for (int g0 = 0; g0 < G; g0 += gh) {
    vector_shape g = s;
    g.n_q_heads = s.n_kv_heads * (g0 + gh <= G ? gh : G - g0);
    // the last group's second pass sees the finished mass: it leaves its statistics for the routing's buckets
    float4* range = (route_ws && g0 + gh >= G) ? reinterpret_cast<float4*>(route_mass_range(route_ws, s.n_kv_heads)) : nullptr;
    const int rc = run_passes<T, D>(stack, s, g, g0 * s.window, g0 > 0, q, k, v, W, true, g0 == 0 ? eps : nullptr, ws, stream, rope,
                                    lse, range, &n_range, &mass, &n_prefix);
    if (rc != VECTOR_OK) return rc;
  }
  if (leave_mass) return VECTOR_OK;
  return launch_pool_scores(mass, score, eps, s.n_kv_heads, s.seq_len, n_prefix, s.pool_kernel, s.pool_mode, route_ws, n_range, stream);
}

template <typename T, int D>
static int run_residual_probe(const vector_shape& s, const void* k, const void* v, const void* W, float* eps, int repeat,
                              hipStream_t stream) {
  PassLaunch L;
  const int rc = prepare_passes<T, D>(nullptr, s, s, 0, false, nullptr, k, v, W, false, eps, nullptr, nullptr, nullptr, nullptr, 0, L);
  if (rc != VECTOR_OK) return rc;
  L.pp.repeat = repeat;
  return launch_probe<T, D>(L, stream);
}

int launch_residual_probe(const vector_shape& s, const void* k, const void* v, const void* W, float* eps, int repeat,
                          hipStream_t stream) {
  if (s.dtype != VECTOR_BF16) return VECTOR_ERR_DTYPE;
  if (s.head_dim == 128) return run_residual_probe<bf16_t, 128>(s, k, v, W, eps, repeat, stream);
  if (s.head_dim == 64) return run_residual_probe<bf16_t, 64>(s, k, v, W, eps, repeat, stream);
  return VECTOR_ERR_SHAPE;
}

int launch_score_residual(const vector_shape& s, const void* q, const void* k, const void* v, const void* W,
                          float* score, float* eps, void* ws, hipStream_t stream, const RopeParams* rope,
                          void* route_ws, const SeqStack* stack, const QueryLse* lse, bool leave_mass) {
  if (s.dtype == VECTOR_BF16) {
    if (s.head_dim == 128) return run_score_residual<bf16_t, 128>(stack, s, q, k, v, W, score, eps, ws, stream, rope, route_ws, lse, leave_mass);
    if (s.head_dim == 64) return run_score_residual<bf16_t, 64>(stack, s, q, k, v, W, score, eps, ws, stream, rope, route_ws, lse, leave_mass);
  } else if (s.dtype == VECTOR_F32) {
    if (s.head_dim == 128) return run_score_residual<float, 128>(stack, s, q, k, v, W, score, eps, ws, stream, rope, route_ws, lse, leave_mass);
    if (s.head_dim == 64) return run_score_residual<float, 64>(stack, s, q, k, v, W, score, eps, ws, stream, rope, route_ws, lse, leave_mass);
  } else {
    return VECTOR_ERR_DTYPE;
  }
  return VECTOR_ERR_SHAPE;
}

bool score_heads_in_one_group(const vector_shape& s) {
  const int G = s.n_q_heads / s.n_kv_heads;
  if (s.dtype == VECTOR_BF16) return s.head_dim == 128 ? heads_per_group<bf16_t, 128>(s) == G : heads_per_group<bf16_t, 64>(s) == G;
  return s.head_dim == 128 ? heads_per_group<float, 128>(s) == G : heads_per_group<float, 64>(s) == G;
}

size_t score_ragged_table_bytes(int count) { return align_up(sizeof(PassParams) * count, 256); }
size_t ragged_table_bytes(int count) {
  return score_ragged_table_bytes(count) + std::max(route_ragged_table_bytes(count), route_head_table_bytes(count));
}

int launch_score_residual_ragged(const vector_shape& s, const RaggedSeq* seqs, int count, const void* W, void* tables,
                                 hipStream_t stream, const RopeParams* rope, bool leave_mass) {
  if (s.dtype == VECTOR_BF16) {
    if (s.head_dim == 128) return run_score_residual_ragged<bf16_t, 128>(s, seqs, count, W, tables, stream, rope, leave_mass);
    if (s.head_dim == 64) return run_score_residual_ragged<bf16_t, 64>(s, seqs, count, W, tables, stream, rope, leave_mass);
  } else if (s.dtype == VECTOR_F32) {
    if (s.head_dim == 128) return run_score_residual_ragged<float, 128>(s, seqs, count, W, tables, stream, rope, leave_mass);
    if (s.head_dim == 64) return run_score_residual_ragged<float, 64>(s, seqs, count, W, tables, stream, rope, leave_mass);
  } else {
    return VECTOR_ERR_DTYPE;
  }
  return VECTOR_ERR_SHAPE;
}

}  // namespace vec
