// Internal interface between the host library (pced_api.cpp) and the gfx950
// kernels (pced_kernels.hip). Not installed; the public ABI is include/pced.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace pced {

constexpr int kPage = 16;          // tokens per KV page (= MFMA M/K tile edge)
constexpr int kMaxGroup = 16;      // q-heads per kv-head (MFMA N edge)
constexpr int kFuseBlock = 256;    // threads of the fuse work-groups
constexpr int kFuseInlineQueries = 32;  // queries whose row offsets the fuse gets in its kernel arguments
constexpr int kBetaChunk = 4096;   // vocab entries per beta work-group
constexpr int kBetaFoldMax = 1024; // experts of a query whose beta the fuse sums itself (LDS)
constexpr int kAggSlice = 256;     // vocab entries per MoE / PoE work-group, or wave
constexpr int kAggExperts = 256;   // experts whose coefficients it holds in LDS at a time
constexpr int kLmRowsPad = 48;     // hidden-state rows are padded to a multiple of this
constexpr int kLmRowsMTW = 9;      // many-row LM head: row tiles per wave (up to 32 * 9 = 288 rows at once)
constexpr int kMaxSplitPages = 64; // pages per attention chunk (one page id per lane)
constexpr int kMaxSeg = 8;         // sequences one decode attention chunk may span (a prefill chunk: one per page)
constexpr int kStageUnits = 4;     // 16-byte q units per lane staged in LDS for a chunk's later sequences
// Packed LM-head tiles ordered [64-wide k step][16-row vocab block]: at every k
// step the waves of a launch read adjacent tiles, so the weight stream sweeps W
// as one front (the fastest HBM read pattern measured) instead of one region per
// wave ([vocab block][k step]).
constexpr bool kLmKMajor = true;
// The decoder projections' packed matrices in the same k-step-major order:
// [64-wide k step][16-column tile], so the blocks working on one K slice read
// adjacent tiles at every step.
constexpr bool kProjKMajor = true;

// Element offsets inside a bf16 KV tile (16 tokens x head_dim; see pced.h, pool
// layout): every matrix-core operand of the attention is one contiguous 16-byte
// load per lane. K token t, dim d: the A operand of the 16x16x32 q.k product;
// V: the A operand of the 16x16x16 V^T.P^T product.
__device__ inline int kswz(int t, int d) {
  return ((d >> 5) * 64 + t + 16 * ((d & 31) >> 3)) * 8 + (d & 7);
}
__device__ inline int vswz(int t, int d) {
  const int j = d >> 4;
  return (((j >> 1) * 64 + (d & 15) + 16 * (t >> 2)) * 2 + (j & 1)) * 4 + (t & 3);
}

// Attention launch arguments: launch_layers layers from `layer` on.
struct AttnArgs {
  const void* q;            // [S][L][Hq][D]
  const void* kpool;        // [L][max_pages][Hkv][tile]
  const void* vpool;
  const int32_t* len0;      // [S] lengths at load
  const int32_t* page_table;// [S][maxpps]
  // Balanced plan of the step (written by the planning blocks of the append
  // launch): the pages of all sequences, concatenated in sequence order, are cut
  // into C chunks of equal size (+-1 page); one wave per (chunk, kv-head). A
  // chunk meets up to kMaxSeg sequences ("segments"; in the prefill up to
  // kMaxSplitPages, of which nothing is staged in advance); each segment yields one
  // partial state of its sequence, or the final output when the sequence lies
  // in a single chunk.
  const int2* chunk_info;   // [C] (segments, pages) of each chunk
  const int4* seg;          // [C][kMaxSeg, prefill kMaxSplitPages][2]: {s, first page in chunk, page offset in s - first page,
                            //  token end in this chunk}, {partial index in s, partials of s, tokens of s, 0}
  const int32_t* nparts;    // [S] partial states of each sequence (chunks it meets)
  const int32_t* work_pages;// [C][kMaxSplitPages] physical pages of each chunk
  float* part_acc;          // [S*Hkv][split_stride][G][D] partial outputs (bf16 path: normalised, as bf16)
  float* part_ml;           // [S*Hkv][split_stride][G][2] (running max in log2 units, sum)
  void* x_out;              // [S][Hq*D] layer output, storage type (null: not wanted)
  float* attn_out;          // optional [S][L][Hq][D]
  float* hidden_out;        // optional [S][Hq*D] (last layer only)
  int launch_layers, n_chunks;             // layers of this launch; chunks C of the plan
  size_t acc_layer_bytes, ml_layer;        // partial states: bytes of part_acc and floats of part_ml per layer
  int x_last_only;          // x_out receives the last layer's output alone (the kernel sets is_last_layer)
  int n_seqs, n_layers, layer, n_q_heads, n_kv_heads, group;
  int max_pages, maxpps, t, split_stride, is_last_layer;
  int kv_reread;            // prefill (k_attn_prefill): pages are read by several token groups
  // prefill only: a sequence's tq_T tokens of the chunk (rows s * tq_T + i) in
  // groups of tq, and `group` counts a token group's tq x (Hq / Hkv) query
  // columns per kv-head; partial states per (sequence, token group)
  int tq, tq_T;
  float scale_log2;         // log2(e) / sqrt(D)
};

struct AppendArgs {
  const void* k_new;        // [S][L][Hkv][D]
  const void* v_new;
  void* kpool;
  void* vpool;
  const int32_t* len0;
  const int32_t* page_table;
  int2* chunk_info;         // plan outputs, see AttnArgs
  int4* seg;
  int32_t* nparts;
  int32_t* work_pages;
  int n_seqs, n_layers, n_kv_heads, head_dim, max_pages, maxpps, t;
  int n_chunks, total_pages;  // C and P of the balanced plan (P = pages after the append)
  int seg_stride;             // segment descriptors per chunk
};

struct LoadArgs {
  const uint64_t* src_k;    // [S] device pointers to [L][len][Hkv][D]
  const uint64_t* src_v;
  const int32_t* items;     // [n_items][2] (sequence, logical page)
  const int32_t* len0;
  const int32_t* page_table;
  void* kpool;
  void* vpool;
  int n_layers, n_kv_heads, head_dim, max_pages, maxpps;
  // items null: n_items consecutive pages of sequence one_s from page0 on, into
  // layers layer0 .. layer0 + n_layers - 1, from rows [n_layers][one_len][Hkv][D]
  // at one_k / one_v that start at token 16 page0
  int n_items;              // (set by launch_load)
  int layer0, one_s, page0, one_len;
  const void* one_k;
  const void* one_v;
};

constexpr int kLmWideMaxRows = 288;  // rows of the largest many-row tile count
constexpr int kLmMaxGroups = 16;     // row groups of the fused many-row LM head

// Row groups of the many-row LM head: every block takes the rows of one group
// (at most 32 mth) against 256 vocabulary rows. groups 0: another kernel runs.
struct LmWidePlan {
  int groups = 0, rows = 0, mth = 0;
  // with the fused epilogue and several groups: the groups' first rows and queries
  int row0[kLmMaxGroups + 1] = {}, q0[kLmMaxGroups + 1] = {};
};

struct LmArgs {
  const void* x;            // [rows_pad][K] storage type, rows >= M zero
  const void* w;            // packed bf16 tiles (see pced_pack_lm_head) or f32 [V][K]
  float* logits;            // [M][V]
  int M, V, K, rms;
  int row_groups;           // >= 1: work-groups per vocab chunk: each takes every R-th 48-row group, or
                            // (many-row kernel) one group of the plan
  int grp_rows;             // rows of an unfused many-row group; the fused ones' first rows and queries:
  int grp_row0[kLmMaxGroups + 1], grp_q0[kLmMaxGroups + 1];
  const LmWidePlan* wide_plan;  // host: the fused launch's row groups when M > 288
  // Fused Eq. 2 epilogue (fuse_part != nullptr; M <= 288 or wide_plan): the
  // logits are not written; every block writes its best two tokens per query
  // (over its vocabulary slice) to fuse_part [B][fuse_nblk][5] for k_fuse_final.
  const int32_t* query_seq0;// [B+1]
  const int32_t* query_exp0;// [B+1]
  const float* beta;        // [sum N]
  const float* prior;       // [sum N]
  const int32_t* exp_seq;   // [sum N] row of each expert (the many-row kernel stages beta and prior by row)
  float* fuse_part;
  int n_queries, fuse_nblk;
  const float* rho_in;      // optional [M] row scales used instead of rms (bf16 kernels)
  float* rho_buf;           // optional [M] scratch: the many-row kernel computes the row scales there first
  void* x_packed;           // optional scratch of lmhead_packed_rows(plan) rows of K bf16: the many-row
                            // kernel's operand-ordered copy of x
  size_t w_vb, w_ks;        // packed W: 16-byte units from one vocab block / 64-wide k step to the next
                            // (set by launch_lmhead from kLmKMajor)
};

struct FuseArgs {
  const float* logits;      // [S][V]
  const int32_t* query_seq0;// [B+1]
  const int32_t* query_exp0;// [B+1]
  const float* beta;        // [sum N]
  const float* prior;       // [sum N] gamma * ln(clip(r)) rounded to fp32
  float* part;              // [B][nblk][5]
  int32_t* tokens_out;      // [B] with stride
  int32_t* prev_tok;        // [B]
  int32_t* winner;          // optional [B]
  float* top1;              // optional [B]
  float* top2;              // optional [B]
  float* beta_used;         // optional [sum N]: beta as used
  int V, nblk, tok_stride;
  int max_n;                // most experts of any query (load batch of the stand-alone fuse)
  // optional: beta is summed from the divergence's chunk partials [sum N][nchunk]
  // (max_n <= kBetaFoldMax) and stored to beta_out
  const float* jsd_part;
  float* beta_out;
  int nchunk;
  int32_t inl_seq0[kFuseInlineQueries + 1];  // query_seq0 / query_exp0 of the first queries
  int32_t inl_exp0[kFuseInlineQueries + 1];
};

// MoE / PoE aggregation (the alternatives to Eq. 3's max): per-expert
// log-sum-exp of the contrastive logits c_k = (1 + beta_k) s_k - beta_k s_0,
// then per vocabulary slice the aggregated score and its best two tokens.
struct AggArgs {
  const float* logits;      // [S][V]
  const int32_t* query_seq0;// [B+1]
  const int32_t* query_exp0;// [B+1]
  const int32_t* exp_seq;   // [sum N]
  const int32_t* exp_query; // [sum N]
  const float* beta;        // [sum N]
  const float* logw;        // [sum N] log pi_k, pi_k = r_k^gamma / sum_j r_j^gamma within the query
  const float* jsd_part;    // optional [sum N][nchunk]: beta is summed from these and stored to beta_out
  float* beta_out;
  float* lse_part;          // [sum N][nchunk][2]
  float* part;              // [B][nblk][5] slice candidates for k_fuse_final (agg_slice() tokens each)
  int V, nchunk, nblk, product;  // product: 0 = mixture (MoE), 1 = product (PoE)
};

struct BetaArgs {
  const float* logits;      // [S][V]
  const int32_t* query_seq0;
  const int32_t* exp_seq;   // [sum N] sequence of each expert slot
  const int32_t* exp_query; // [sum N] query of each expert slot
  float* lse_part;          // [S][nchunk][2]
  float* jsd_part;          // [sum N][nchunk]
  float* beta;              // [sum N]
  const int32_t* query_exp0;// [B+1] (scalar mode)
  int V, nchunk;
};

struct SynthArgs {
  void* q;                  // [S][L][Hq*D]
  void* k_new;              // [S][L][Hkv*D]
  void* v_new;
  const int32_t* seq_query; // [S]
  const int32_t* prev_tok;  // [B]
  uint64_t seed;
  float value_scale;        // sqrt(3)/65536 rounded to fp32
  int n_layers, qdim, kvdim, t, first_token, use_first, bf16;
};

// Decoder-stack projections of one decode step: out[m][n] = rho_m sum_k x[m][k] W[n][k]
// for the M step rows, W packed in 16-row tiles (k_pack_w_bf16 layout), with an
// epilogue per projection.
enum GemmEpi { kEpiQkv = 0, kEpiResid = 1, kEpiSwiglu = 2 };
// Rows of the projection kernels; more go to the library GEMM. Per layer (QKV, O, gate/up, down),
// kernel / library: Llama-3-8B shapes 49 rows 105 / 142 us, 97 rows 136 / 166, 128 rows 153 / 204; hidden
// 3584, MLP 18944: 49 rows 129 / 200, 128 rows 186 / 239; hidden 512, MLP 1408: 128 rows 58 / 107. Eight
// row tiles are what the rings' 128 KiB of LDS hold; 129 rows take the library 193 us (Llama-3-8B).
constexpr int kProjMaxRows = 128;
constexpr int kProjMaxSplit = 16;  // K slices of a projection (partial buffer sized for this many)
constexpr int kPrefillRows = 2304;  // (sequence, suffix token) rows of one prefill chunk, at least
constexpr int kPrefillTiles = 2;   // 16-column query tiles of a prefill token group, at most
constexpr int kPrefillWaves = 8;   // waves per compute unit, and at most per block, of the prefill attention (its registers)
constexpr int kPrefillParts = 8;   // attention partial states per prefill row and kv-head
struct GemmArgs {
  const void* w;            // packed tiles of this projection
  const uint16_t* x;        // [M][K] bf16 input rows
  int M, K, n_tiles;        // rows, inner dimension, 16-column output tiles
  int ksplit;               // K slices (blocks per column group)
  float* part;              // [ksplit][M][16 n_tiles] fp32 partial sums
  // row scale rho_m = 1/sqrt(sum_p ss_in[p][m] * inv_norm_dim + eps), or 1 without ss_in
  const float* ss_in;       // [M][ld_ss]: row m's per-16-column sums at m * ld_ss + p, p < ss_parts
  // many-row epilogues (launch_proj_epilogue): [M] scratch that receives the row
  // scales of ss_in once (k_rho), read as rho_in instead of a sum in every block
  float* rho_rows;
  const float* rho_in;
  int ss_parts, ld_ss;
  float inv_norm_dim, eps;
  // kEpiResid: h[m][n] += out; a_out = bf16(h * g_next); ss_out[n / 16][m] = sum of h^2 over the tile
  float* h;                 // [M][hidden]
  uint16_t* a_out;          // [M][hidden]
  const uint16_t* g_next;   // [hidden]
  float* ss_out;            // [rows][ld_ss], ld_ss >= hidden/16
  // kEpiSwiglu: tiles alternate gate / up; act[m][f] = bf16(silu(gate) * up)
  uint16_t* act;            // [M][F]
  int F;
  // kEpiQkv: columns [0, Hq*D) q, then k, then v; RoPE at pos = len0[m] + t;
  // q to q_out, k / v into the paged pool at that position
  uint16_t* q_out;          // [S][L][Hq][D]
  uint16_t* qkv_trace;      // optional [M][Hq*D + 2 Hkv*D]: q, k, v after RoPE as stored (parity tracing)
  uint16_t* kpool;
  uint16_t* vpool;
  const int32_t* len0;
  const int32_t* page_table;
  int layer, n_layers, n_q_heads, n_kv_heads, head_dim, max_pages, maxpps, t;
  double log2_theta;
  // [maxpps * page][head_dim / 2]: (cos, sin) of RoPE angle pos * theta^(-2i/D)
  // for each position and pair i (launch_rope_table)
  const float2* rope;
};
struct EmbedArgs {
  const uint16_t* embed;    // [V][hidden]
  const uint16_t* g;        // [hidden] first layer's attention norm weight
  const int32_t* tokens;    // [B] with stride
  const int32_t* seq_query; // [S]
  float* h;                 // [S][hidden]
  uint16_t* a_out;          // [S][hidden] bf16(h * g)
  float* ss_out;            // [rows][ld_ss], ld_ss >= hidden/16
  int hidden, vocab, tok_stride, ld_ss;
};
// Rows of one prefill chunk: row r = s*T + i is sequence s's suffix token i0 + i,
// a virtual sequence over s's pages ending at position len_s + i. For the
// attention's plan (tq = T) there is one row per sequence, ending at its last token.
struct PrefillMetaArgs {
  const int32_t* len0;      // [S]
  const int32_t* page_table;// [S][maxpps]
  const int32_t* seq_query; // [S]
  int32_t* len0_out;        // [rows] len0[s] + i
  int32_t* page_table_out;  // [rows][maxpps] copy of s's row
  int32_t* tok_map;         // [S*T] index of the row's token in tokens [B][n_tokens] (optional)
  int n_seqs, T, i0, n_tokens, maxpps;
  int tq;                   // >= 1: one output row per group of tq tokens (len0 of its last token)
};
// Copy of tokens [start, start + count) of one sequence and layer out of the pool.
struct ReadCacheArgs {
  const void* kpool;
  const void* vpool;
  const int32_t* page_table;  // device [S][maxpps]
  void* k_out;                // [count][Hkv][D]
  void* v_out;
  int seq, layer, start, count, n_kv_heads, head_dim, max_pages, maxpps, bf16;
};

// Optional timing events attached to the first / last dispatch of a launcher.
struct Timing {
  hipEvent_t start = nullptr;
  hipEvent_t stop = nullptr;
};

// launchers (pced_kernels.hip); each returns hipGetLastError() after the launch
hipError_t launch_fill_i32(int32_t* p, int32_t v, size_t n, hipStream_t st);
hipError_t launch_zero_bytes(void* p, size_t nbytes, hipStream_t st);
hipError_t launch_load(const LoadArgs& a, int n_items, bool bf16, hipStream_t st, const Timing* tm = nullptr);
hipError_t launch_append(const AppendArgs& a, bool bf16, hipStream_t st, const Timing* tm = nullptr);
hipError_t launch_attn(const AttnArgs& a, int head_dim, bool bf16, hipStream_t st, const Timing* tm = nullptr);
int attn_blocks_per_cu(int head_dim, bool bf16);  // resident one-wave blocks per CU
hipError_t launch_attn_combine(const AttnArgs& a, int head_dim, bool bf16, hipStream_t st, const Timing* tm = nullptr);
hipError_t launch_pack_lm_head(const void* w, void* wp, int V, int K, bool bf16, hipStream_t st);
hipError_t launch_lmhead(const LmArgs& a, bool bf16, hipStream_t st, const Timing* tm = nullptr);
// the divergence's chunk partials, and with `sums` beta itself
hipError_t launch_beta(const BetaArgs& a, int n_seqs, int n_exp, bool sums, hipStream_t st, const Timing* tm = nullptr);
// k_fuse (timed by tm) then the per-query merge k_fuse_final (timed by tm_merge)
hipError_t launch_fuse(const FuseArgs& a, int n_queries, hipStream_t st, const Timing* tm = nullptr,
                       const Timing* tm_merge = nullptr);
// vocabulary tokens per work-group of the stand-alone fuse (1024, or 512 for few queries)
int fuse_slice(int V, int n_queries, int num_cus);
// vocabulary tokens per work-group of the MoE / PoE aggregation (kAggSlice, or 4 kAggSlice for many
// queries of few experts); max_n: most experts of any query
int agg_slice(int V, int n_queries, int max_n, int num_cus);
hipError_t launch_beta_mean(const BetaArgs& a, int n_queries, hipStream_t st);
hipError_t launch_agg(const AggArgs& a, int n_exp, int n_queries, hipStream_t st, const Timing* tm = nullptr);
// the final per-query merge alone (after an LM head with the fused epilogue)
hipError_t launch_fuse_final(const FuseArgs& a, int n_queries, hipStream_t st, const Timing* tm = nullptr);
// vocabulary slices (blocks) of the fused LM-head epilogue for M rows, or 0 if M
// rows cannot be fused (groups: a plan of query-aligned row groups is given)
int lmhead_fused_nblk(int M, int V, bool groups = false);
// Row groups of the many-row LM head for M rows of a bf16 LM head, or none if
// another kernel runs; for the fused epilogue of more than 288 rows, groups of
// whole queries (seq_off [n_queries + 1]: the queries' first rows) whose packed x
// takes at most max_packed_rows rows, or none
LmWidePlan lmhead_wide_plan(int M, int V, int K);
LmWidePlan lmhead_wide_plan_queries(const int32_t* seq_off, int n_queries, int V, int K, int max_packed_rows);
size_t lmhead_packed_rows(const LmWidePlan& p);  // rows of the plan's packed x (padded tiles included)
hipError_t launch_synth(const SynthArgs& a, int n_seqs, hipStream_t st, const Timing* tm = nullptr);
hipError_t launch_copy_rows(const void* src, void* dst, size_t nbytes, hipStream_t st);
hipError_t launch_stream_read(const void* src, size_t nbytes, uint32_t* xor_out, int num_cus, hipStream_t st);
// pack a [rows][K] bf16 matrix into 16-row tiles, tile i going to slot i * stride + offset
hipError_t launch_pack_tiles(const void* w, void* wp, int rows, int K, int stride, int offset, int n_tiles,
                             hipStream_t st);
hipError_t launch_gemm(const GemmArgs& a, GemmEpi epi, hipStream_t st, const Timing* tm = nullptr);
// The projection epilogue alone, over products already in a.part as one K
// slice ([M][16 n_tiles] fp32, e.g. from a library GEMM).
hipError_t launch_proj_epilogue(const GemmArgs& a, GemmEpi epi, hipStream_t st, const Timing* tm = nullptr);
int proj_ksplit(int n_tiles, int K, int num_cus);  // K slices of a projection of at most kProjMaxRows rows
hipError_t launch_embed(const EmbedArgs& a, int n_seqs, hipStream_t st, const Timing* tm = nullptr);
hipError_t launch_prefill_meta(const PrefillMetaArgs& a, hipStream_t st);
// rho[m] = 1/sqrt(sum_p ss[p][m] * inv_dim + eps) for m < M
hipError_t launch_read_cache(const ReadCacheArgs& a, hipStream_t st);
// The allocation-free entry point's scratch: a library-owned device array of
// kNoAllocScratchBytes per GPU; out = its address on the current device.
constexpr size_t kNoAllocScratchBytes = (size_t)4 << 20;
hipError_t noalloc_scratch(void** out);
hipError_t launch_rho(const float* ss, int parts, int ld, int M, float inv_dim, float eps, float* rho,
                      hipStream_t st);
// RoPE table of GemmArgs::rope for positions 0 .. positions - 1, in fp64 rounded to fp32
hipError_t launch_rope_table(float2* out, int positions, int head_dim, double log2_theta, hipStream_t st);

}  // namespace pced
