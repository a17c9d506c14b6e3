// Integer kernels of the verification step: the majority vote over SSM drafts (paper section 3.2,
// "Tree-based Weighted Majority Decision"), longest-prefix acceptance with KV commit (section
// 2.1 in its greedy case; section 4 for the deletion of rejected tokens' cache entries), and the
// speculation quality metric with the SSM weight update that closes the loop (section 3.2,
// equation ACR).
#include "launch.h"
#include "../../include/minions_verify.h"

namespace mn {

// One wave per sequence, lane j = draft j (n <= 64).  The token tree is never materialised: `alive` is the set of drafts
// whose prefix equals the path chosen so far, which is exactly the subtree below the current node.  A child's
// weight is accumulated in fp32 in ascending draft order (the order is part of the result): every lane adds up
// the weights of the drafts that hold its own token.  The drafts of eight levels are asked for at once; with one
// thread per sequence every level was a chain of dependent loads (64 sequences x 5 drafts x 16 tokens: 14.8 us, now 5.5).
__global__ void __launch_bounds__(256) vote_kernel(const int32_t* __restrict__ drafts, const int32_t* __restrict__ spec_len,
                                                   const float* __restrict__ ssm_w, int B, int n, int k_max, int mode,
                                                   int32_t* __restrict__ voted, int32_t* __restrict__ voted_ssm,
                                                   int32_t* dev_status) {
  constexpr int CHUNK = 8;
  const int b = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (b >= B) return;  // (whole wave)
  const int32_t* D = drafts + (size_t)b * n * k_max + (size_t)min(lane, n - 1) * k_max;
  int32_t* out = voted + (size_t)b * k_max;
  const int k = spec_len[b];
  if (k < 0 || k > k_max) {
    if (dev_status && lane == 0) atomicOr(dev_status, MN_DEV_DRAFTS);
    for (int t = lane; t < k_max; t += 64) out[t] = -1;
    if (lane == 0) voted_ssm[b] = -1;
    return;
  }
  const float w = ssm_w[min(lane, n - 1)];
  const uint64_t all = (n >= 64) ? ~0ull : ((1ull << n) - 1ull);
  uint64_t alive = all;  // drafts equal to the result so far
  for (int t0 = 0; t0 < k; t0 += CHUNK) {
    int tok[CHUNK];
#pragma unroll
    for (int u = 0; u < CHUNK; ++u) tok[u] = D[min(t0 + u, k - 1)];
#pragma unroll
    for (int u = 0; u < CHUNK; ++u) {
      if (t0 + u >= k) break;
      const uint64_t pool = (mode == MN_VOTE_TREE) ? alive : all;
      float W = 0.f;
      for (uint64_t rest = pool; rest; rest &= rest - 1) {
        const int j = __ffsll((unsigned long long)rest) - 1;
        const float wj = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), j));
        if (__builtin_amdgcn_readlane(tok[u], j) == tok[u]) W += wj;
      }
      // heaviest token of the pool; of equal ones the first supported (a draft repeating an earlier one's token has its
      // weight and never exceeds it)
      int best_tok = -1;
      float best_w = 0.f;
      bool have = false;
      for (uint64_t rest = pool; rest; rest &= rest - 1) {
        const int j = __ffsll((unsigned long long)rest) - 1;
        const float Wj = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, W), j));
        if (!have || Wj > best_w) {
          have = true;
          best_w = Wj;
          best_tok = __builtin_amdgcn_readlane(tok[u], j);
        }
      }
      if (lane == 0) out[t0 + u] = best_tok;
      alive &= __ballot(lane < n && tok[u] == best_tok);
    }
  }
  for (int t = k + lane; t < k_max; t += 64) out[t] = -1;
  if (lane == 0) voted_ssm[b] = __ffsll((unsigned long long)alive) - 1;  // (none: -1)
}

void launch_vote(const int32_t* drafts, const int32_t* spec_len, const float* ssm_w, int B, int n, int k_max, int mode,
                 int32_t* voted, int32_t* voted_ssm, int32_t* dev_status, hipStream_t st) {
  if (B <= 0) return;
  vote_kernel<<<(B + 3) / 4, 256, 0, st>>>(drafts, spec_len, ssm_w, B, n, k_max, mode, voted, voted_ssm, dev_status);
}

// One wave per sequence: longest matching prefix, emitted tokens, context advance.
__global__ void __launch_bounds__(256) accept_commit_kernel(const int32_t* __restrict__ voted, const int32_t* __restrict__ greedy,
                                     const int32_t* __restrict__ spec_len, int B, int k_max, int32_t* ctx_lens,
                                     int block_size, int max_blocks_per_seq, int32_t* __restrict__ accepted_len,
                                     int32_t* __restrict__ out_tokens, int32_t* __restrict__ n_out,
                                     int32_t* __restrict__ next_last_tok, int32_t* __restrict__ blocks_in_use,
                                     int32_t* dev_status) {
  const int b = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (b >= B) return;  // (whole wave)
  const int32_t* g = greedy + (size_t)b * (k_max + 1);
  int32_t* o = out_tokens + (size_t)b * (k_max + 1);
  const int k = spec_len[b];
  const int ctx = ctx_lens[b];
  const int g0 = g[0];
  bool ok = (k >= 0 && k <= k_max && g0 >= 0);
  if (lane == 0 && (k < 0 || k > k_max)) {
    if (dev_status) atomicOr(dev_status, MN_DEV_SPEC_LEN);
  }
  int a = 0;
  if (ok) {
    const int32_t* v = voted + (size_t)b * k_max;
    for (; a < k; a += 64) {             // 64 positions at a time; the first that differs ends the prefix
      const int t = a + lane;
      const uint64_t differ = __ballot(t < k && v[min(t, k - 1)] != g[min(t, k - 1)]);
      if (differ) {
        a += __ffsll((unsigned long long)differ) - 1;
        break;
      }
    }
    a = min(a, k);
    const long cap = (long)max_blocks_per_seq * block_size;
    if ((long)ctx + a + 1 > cap) {
      ok = false;
      if (lane == 0 && dev_status) atomicOr(dev_status, MN_DEV_BLOCK_TABLE);
    }
  }
  for (int t = lane; t <= k_max; t += 64) o[t] = (ok && t <= a) ? g[t] : -1;
  if (lane != 0) return;
  const int nc = ok ? ctx + a + 1 : ctx;
  accepted_len[b] = ok ? a : 0;
  n_out[b] = ok ? a + 1 : 0;
  next_last_tok[b] = ok ? g[a] : -1;
  if (ok) ctx_lens[b] = nc;
  blocks_in_use[b] = (nc + block_size - 1) / block_size;
}

void launch_accept_commit(const int32_t* voted, const int32_t* greedy, const int32_t* spec_len, int B, int k_max,
                          int32_t* ctx_lens, int block_size, int max_blocks_per_seq, int32_t* accepted_len,
                          int32_t* out_tokens, int32_t* n_out, int32_t* next_last_tok, int32_t* blocks_in_use,
                          int32_t* dev_status, hipStream_t st) {
  if (B <= 0) return;
  accept_commit_kernel<<<(B + 3) / 4, 256, 0, st>>>(voted, greedy, spec_len, B, k_max, ctx_lens, block_size,
                                                    max_blocks_per_seq, accepted_len, out_tokens, n_out, next_last_tok,
                                                    blocks_in_use, dev_status);
}

// Average acceptance rate per SSM and the multiplicative weight update (section 3.2, equation ACR).
// Thread i owns SSM i and walks the batch in ascending order: ACR_i is the mean, in fp64, of
// accepted_len / spec_len over the verified outputs whose voted SSM is i (outputs with nothing
// speculated, or that the step did not verify, are not in the set).  An SSM that won no vote keeps its
// weight and reports NaN.  The sum is sequential, so the result does not depend on the launch.
__global__ void acr_update_kernel(const int32_t* __restrict__ voted_ssm, const int32_t* __restrict__ accepted_len,
                                  const int32_t* __restrict__ spec_len, const int32_t* __restrict__ n_out, int B, int n,
                                  double reward_threshold, double punish_threshold, float reward_factor,
                                  float punish_factor, float* ssm_w, double* __restrict__ acr) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double sum = 0.0;
  int cnt = 0;
  for (int b = 0; b < B; ++b) {
    const int k = spec_len[b];
    if (voted_ssm[b] != i || k <= 0 || (n_out && n_out[b] <= 0)) continue;
    sum += (double)accepted_len[b] / (double)k;
    ++cnt;
  }
  if (cnt == 0) {
    if (acr) acr[i] = __longlong_as_double(0x7ff8000000000000ll);
    return;
  }
  const double r = sum / (double)cnt;
  if (acr) acr[i] = r;
  if (r > reward_threshold) ssm_w[i] = ssm_w[i] * reward_factor;
  else if (r < punish_threshold) ssm_w[i] = ssm_w[i] * punish_factor;
}

void launch_acr_update(const int32_t* voted_ssm, const int32_t* accepted_len, const int32_t* spec_len,
                       const int32_t* n_out, int B, int n, double reward_threshold, double punish_threshold,
                       float reward_factor, float punish_factor, float* ssm_w, double* acr, hipStream_t st) {
  if (n <= 0) return;
  acr_update_kernel<<<1, 64, 0, st>>>(voted_ssm, accepted_len, spec_len, n_out, B, n, reward_threshold, punish_threshold,
                                      reward_factor, punish_factor, ssm_w, acr);
}

}  // namespace mn
