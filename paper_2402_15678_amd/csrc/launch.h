// Internal launchers: one per kernel family.  Host-side shape checks happen in api.hip; the
// launchers assume validated arguments and only translate them into grids.
//
// Leading arguments.  The command processor puts the first 14 dwords of a kernel's arguments into scalar registers before its
// waves start (build.py: -amdgpu-kernarg-preload-count); everything behind them, and every field of a struct wherever it stands,
// is a scalar load whose round trip the first memory access of every launch waits for.  So what a kernel's first addresses are
// made of is passed twice, as leading plain arguments and in its struct, and the kernel writes the former over the latter.
#pragma once
#include "common.h"

namespace mn {

// ---- vote_accept.hip ----
void launch_vote(const int32_t* drafts, const int32_t* spec_len, const float* ssm_w, int B, int n, int k_max, int mode,
                 int32_t* voted, int32_t* voted_ssm, int32_t* dev_status, hipStream_t st);
void launch_acr_update(const int32_t* voted_ssm, const int32_t* accepted_len, const int32_t* spec_len,
                       const int32_t* n_out, int B, int n, double reward_threshold, double punish_threshold,
                       float reward_factor, float punish_factor, float* ssm_w, double* acr, hipStream_t st);
void launch_accept_commit(const int32_t* voted, const int32_t* greedy, const int32_t* spec_len, int B, int k_max,
                          int32_t* ctx_lens, int block_size, int max_blocks_per_seq, int32_t* accepted_len,
                          int32_t* out_tokens, int32_t* n_out, int32_t* next_last_tok, int32_t* blocks_in_use,
                          int32_t* dev_status, hipStream_t st);

// ---- stochastic.hip ----
void launch_verify_sample(const float* logits, const int32_t* voted, const float* draft_probs, const int32_t* spec_len,
                          const int32_t* greedy, int B, int k_max, int M, int V, double temperature, uint64_t seed,
                          uint64_t step, int32_t* sampled, int32_t* dev_status, hipStream_t st);
void launch_draft_sample(const float* logits, int B, int V, double temperature, uint64_t seed, uint64_t step, int ssm,
                         int t_pos, int32_t* tokens, long token_stride, float* probs, long probs_stride, hipStream_t st);
int verify_sample_max_vocab();

// ---- rows.hip ----
// Work list of the attention kernels, written once per step with the row bookkeeping (attention_plan fills this in).
struct AttnPlan {
  int32_t* items;       // [grid_items] records of 8 int32, or null: the kernel that will run needs no list
  int32_t* row_splits;  // [M]
  int grid_items, tiles16_per_wg, n_splits_max;
  int target_wgs;       // workgroups with work to aim for
  int min_tiles;        // fewest key tiles a workgroup should take
};
struct PrepArgs {
  const int32_t *last_tok, *voted, *spec_len, *ctx_lens, *block_tables;
  int B, k_max, M, vocab, max_pos, block_size, num_blocks, max_blocks_per_seq;
  int max_ctx;       // the host's bound on ctx_b + k_b + 1 (it sized the attention launch)
  int max_q;         // the host's largest number of rows of a sequence (likewise)
  int rope_half;     // head_dim/2 for rotary models, 0 otherwise
  float rope_base;
  int32_t *row_seq, *row_j, *row_pos, *row_tok, *row_slot, *seq_row0, *seq_ctx, *seq_ok;
  int kv_heads;                // KV heads of the model (the attention grid has one workgroup row per KV head)
  int q_per_kv;                // query heads per KV head (a workgroup covers 128 rows of query position x head)
  AttnPlan plan;               // the attention work list to write (items null: none)
  float *rope_cos, *rope_sin;  // [M][rope_half]
  int32_t* dev_status;
};
// hipSuccess, or the error of a one-time kernel attribute setting that failed (nothing is launched then)
hipError_t launch_prepare(const PrepArgs& a, hipStream_t st);

struct NormArgs {
  // source of the row: either the residual stream x (+ partial sums + bias), or the embeddings
  float* x;               // [M][d] residual stream, updated in place
  const float* partials;  // [S][M][d] or null
  int n_partials;
  const float* bias;      // [d] or null
  const void* tok_emb;    // when non-null the row is tok_emb[row_tok] (+ pos_emb[row_pos])
  const void* pos_emb;
  const int32_t *row_tok, *row_pos;
  const float *gain, *shift;  // shift null => RMSNorm
  float eps;
  void* h;                // [M][d] normalised output in the activation type
  int M, d, dtype;
  int32_t* dev_status;    // MN_DEV_RANGE is OR-ed in when an fp16 output saturates, or null
  float* rstd;            // [M] 1 / rms of the rows, or null
  bool operand;           // h in operand order (common.h)
};
void launch_norm(const NormArgs& a, hipStream_t st);

struct RopeAppendArgs {
  const float* qkv;  // [S][M][(H+2Hkv)*hd] partial sums
  int n_partials;
  const float* bias;  // [(H+2Hkv)*hd] or null
  const float *rope_cos, *rope_sin;  // [M][hd/2] or null (no rotation)
  RowInfo rows;
  KvView kv;
  void* q;  // [M][H][hd] activation type
  int M, H, Hkv, hd, dtype;
  int32_t* dev_status;  // MN_DEV_RANGE is OR-ed in when an fp16 output saturates, or null
};
void launch_rope_append(const RopeAppendArgs& a, hipStream_t st);

// act[m][f] = relu(sum_s p[s][m][f] + b[f])  or  silu(gate) * up with gate = column f, up = column F + f
struct ActArgs {
  const float* partials;  // [S][M][ncols]
  int n_partials;
  const float* bias;
  void* act;  // [M][F] activation type
  int M, F, swiglu, dtype;
  int32_t* dev_status;  // MN_DEV_RANGE is OR-ed in when an fp16 output saturates, or null
};
void launch_act(const ActArgs& a, hipStream_t st);

// partials non-null: the scores are the sums of S partial sums [S][M][V] and are written to logits first
void launch_argmax_rows(float* logits, const float* partials, int S, int M, int V, const RowInfo& rows, int k_max, int32_t* greedy, int B,
                        hipStream_t st);

// ---- gemm.hip ----
struct GemmArgs {
  const void* a;  // [M][K] activation type (fp32 in fp32 models, fp16 in bf16 models)
  const void* w;  // fp32 models: [N][K] row-major; bf16 models: the packed layout of gemm.hip
  float* out;     // [S][M][N] fp32 partial sums (S = split_k); bias added to split 0 when given
  void* swiglu_act;  // non-null: fused SwiGLU epilogue, fp16 [M][N/2] (bf16 models, split_k == 1, interleaved packing)
  void* relu_act;    // non-null: fused bias + ReLU epilogue, activation type [M][N] (split_k == 1)
  const float* bias;
  int M, N, K, split_k, dtype;
  int32_t* dev_status;  // MN_DEV_RANGE is OR-ed in when a fused fp16 epilogue saturates a value, or null
  const NormArgs* norm;  // non-null (fp32 models, gemm_f32_folds_norm): a is this norm's output, computed on the way; the residual
  float* x_new;          // stream norm->x is left as it is and its new values go to x_new
};
bool gemm_f32_folds_norm(int M, int d_model);
bool gemm_small_matrix(int N, int K);  // so few weights that a projection is launch and memory latency
int gemm_pick_split(int M, int N, int K, int dtype);  // the library's choice; sizes the workspace
int gemm_step_split(int M, int N, int K, int dtype, size_t room);
int gemm_tile_rows(int M, int N, int K, int split);
size_t packed_weight_elems(int N, int K);
void launch_pack_weight(const void* src, void* dst, int N, int K, int half, int32_t* status, hipStream_t st);
// hipSuccess, or the error of a one-time kernel attribute setting that failed (nothing is launched then)
hipError_t launch_gemm(const GemmArgs& a, hipStream_t st);
void launch_reduce_partials(const float* partials, int S, size_t stride, float* out, size_t n, hipStream_t st);

// ---- gemm_small.hip ----
enum { SMALL_OUT = 0, SMALL_SWIGLU = 1, SMALL_RESIDUAL = 2 };
struct SmallGemmArgs {
  const void* a;  // fp16 [M][K] in operand order (common.h)
  const void* w;  // packed
  int M, N, K;
  // SMALL_OUT, SMALL_SWIGLU: with ss, row m of a is x * gain / inv_sc[m] and its norm is applied here; ss null: rows are used as they are.
  // SMALL_RESIDUAL writes them for the projection behind it, from the 1 / rms that the one before it left in rstd.
  float* ss;      // [K / 16] (SMALL_RESIDUAL: [N / 16]) [M] sums of squares of 16 columns of x; sign bit: see gemm_small.hip
  float* inv_sc;  // [M]
  float* rstd;    // [M] 1 / rms of the rows
  int ss_tiles;
  float inv_d, eps;
  float* x;           // residual stream, K (SMALL_RESIDUAL: N, updated in place) columns
  const float* gain;  // of the norm
  void* out;          // SMALL_OUT: fp32 [M][N]; SMALL_SWIGLU: fp16 [M][N / 2], SMALL_RESIDUAL: fp16 x * gain / inv_sc, both in operand order
  int32_t* dev_status;
};
bool gemm_small_model(int M, int n_qkv, int d_model, int hdim, int w1_rows, int d_ffn);
void launch_gemm_small(const SmallGemmArgs& a, int mode, hipStream_t st);

// ---- attention.hip ----
struct AttnArgs {
  const void* q;  // [M][H][hd] activation type
  void* out;      // [M][H*hd] activation type
  bool operand;   // out in operand order (common.h): only where attention_fuses_append
  RowInfo rows;
  KvView kv;      // every key is read from the pages, this step's own (appended before the call) included
  int B, M, H, Hkv, hd, dtype, max_ctx;
  int max_q;       // largest number of rows of one sequence (host knowledge)
  float* scratch;  // split-KV partials
  size_t scratch_bytes;
  int32_t* items;        // work list of the MFMA kernel, 8 int32 per record (see prepare_kernel), or null
  size_t items_capacity; // records the buffer holds
  int32_t* row_splits;   // [M] KV splits of the row's sequence (written by the plan, read by the merge), or null
  bool append;           // this step's rows are still to be turned and appended, in the kernel or by a launch before it
  // Rotary embedding and KV append inside the attention kernel (attention_fuses_append): the QKV projection's partial
  // sums as in RopeAppendArgs; q is not read then.  qkv null: q holds the queries and the pages hold every row.
  const float* qkv;      // [S][M][(H+2Hkv)*hd]
  int n_partials;
  const float* bias;
  const float *rope_cos, *rope_sin;
  int32_t* dev_status;
};
size_t attention_scratch_bytes(int M, int H, int hd, int max_ctx, int dtype);
bool attention_mfma_supported(int H, int Hkv, int hd, int block_size, int dtype);
size_t attention_items_capacity(int B, int M, int H, int Hkv);
bool attention_fuses_append(const AttnArgs& a);  // the kernel that will run can take qkv (needs everything else set)
AttnPlan attention_plan(const AttnArgs& a);  // what the kernels that will run need from the row bookkeeping
// hipSuccess, or the error of a one-time kernel attribute setting that failed (nothing is launched then)
hipError_t launch_attention(const AttnArgs& a, hipStream_t st);

}  // namespace mn
