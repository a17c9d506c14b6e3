// Row-wise kernels of the verification forward: row bookkeeping, embedding + LayerNorm/RMSNorm with
// the residual update folded in, rotary embedding + tentative KV append, FFN activation, vocabulary
// argmax.  The paper (section 4) only states that every scored token's cache entry is addressed
// by a logical block id and an offset; the decoder body is the standard pre-norm one.
#include "launch.h"
#include "../../include/minions_verify.h"

#include <mutex>

namespace mn {

// ------------------------------------------------------------------------------------------
// prepare: validate the batch on the device, lay out the packed rows, list the attention workgroups, rotary table
// ------------------------------------------------------------------------------------------
// One launch per step.  Workgroup 0 does the bookkeeping and then, from the same LDS arrays, the attention work list (the
// same for every layer); the other workgroups fill the rotary table beside it, from the inputs alone (a row's sequence
// and position need only the speculation lengths and contexts).  Bound by dependent round trips, so every table is
// walked by all threads side by side.  Three launches before; 845 prompt rows in 3 sequences took 100 us when a thread
// laid out a whole sequence's rows (120 us with the other two launches, 9.9 now; 618 rows of 64 sequences 32 -> 15, 144 of 16
// 17 -> 9).
constexpr int PREP_THREADS = 1024;
constexpr int RANK_WAVES = 64;   // most sequences whose place in the attention work list is found by a wave each
template <int N> struct IntC { static constexpr int value = N; };

// s_row0[b] = first row of sequence b (b = 0 .. B), from s_row0[b + 1] = rows of sequence b.  Every thread of the workgroup.
__device__ __forceinline__ void scan_rows(int32_t* s_row0, int B, int32_t* s_wave) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (B <= 64) {                            // one wave holds them all
    if (tid < 64) {
      const int inc = wave_scan_i(tid < B ? s_row0[tid + 1] : 0);
      if (tid < B) s_row0[tid + 1] = inc;
      if (tid == 0) s_row0[0] = 0;
    }
    __syncthreads();
    return;
  }
  const int per = (B + PREP_THREADS - 1) / PREP_THREADS, lo = min(tid * per, B), hi = min(lo + per, B);
  int sum = 0;
  for (int b = lo; b < hi; ++b) sum += s_row0[b + 1];
  const int inc = wave_scan_i(sum);
  if (lane == 63) s_wave[wave] = inc;
  __syncthreads();
  int at = inc - sum;
  for (int w = 0; w < wave; ++w) at += s_wave[w];
  for (int b = lo; b < hi; ++b) {
    at += s_row0[b + 1];
    s_row0[b + 1] = at;
  }
  if (tid == 0) s_row0[0] = 0;
  __syncthreads();
}
// the sequence of row m: largest b with s_row0[b] <= m (every sequence has at least one row)
__device__ __forceinline__ int seq_of_row(const int32_t* s_row0, int B, int m) {
  int lo = 0, hi = B - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (s_row0[mid] <= m) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// cos/sin of the rotary angles, evaluated in double once per step and shared by all layers
__device__ __forceinline__ void rope_rows(const PrepArgs& a, const int32_t* s_row0, const int32_t* s_ctx) {
  const int half = a.rope_half, rows = PREP_THREADS / half;
  const int m = ((int)blockIdx.x - 1) * rows + (int)threadIdx.x / half, i = (int)threadIdx.x % half;
  if (m >= a.M || (int)threadIdx.x >= rows * half) return;
  const int b = seq_of_row(s_row0, a.B, m);
  const int p = s_ctx[b] + m - s_row0[b];  // (the rows of a disabled sequence are never used)
  const double inv = pow((double)a.rope_base, -2.0 * (double)i / (double)(2 * half));
  const double ang = (double)p * inv;
  a.rope_cos[(size_t)m * half + i] = (float)cos(ang);
  a.rope_sin[(size_t)m * half + i] = (float)sin(ang);
}

// LDS: six int32 arrays of B + 1 entries
__global__ void __launch_bounds__(PREP_THREADS) prepare_kernel(const int32_t* spec_len_, const int32_t* ctx_lens_, const int32_t* block_tables_,
                                                                const int32_t* last_tok_, const int32_t* voted_, int B_, int max_q_,
                                                                int max_blocks_, int k_max_, PrepArgs a) {
  a.spec_len = spec_len_; a.ctx_lens = ctx_lens_; a.block_tables = block_tables_; a.last_tok = last_tok_;  // (launch.h: leading arguments)
  a.voted = voted_; a.B = B_; a.max_q = max_q_; a.max_blocks_per_seq = max_blocks_; a.k_max = k_max_;
  extern __shared__ __attribute__((aligned(16))) int32_t s_prep[];
  __shared__ int32_t s_wave[PREP_THREADS / 64];
  __shared__ int s_bad;
  __shared__ unsigned long long s_tiles;
  const int tid = threadIdx.x, B = a.B;
  int32_t* s_row0 = s_prep;                 // [B + 1]
  int32_t* s_ok = s_row0 + B + 1;           // [B]
  int32_t* s_nb = s_ok + B + 1;             // [B] blocks a sequence needs mapped (0: nothing to check); later tiles per workgroup
  int32_t* s_cnt = s_nb + B + 1;            // [B] attention workgroups of a sequence
  int32_t* s_spl = s_cnt + B + 1;           // [B] its KV splits
  int32_t* s_ctx = s_spl + B + 1;           // [B] context
  // The first loads of every table go out at once, the numbers that the others wait for first: none of them needs another's answer
  // to know its place.  Block table: entry tid + 1024 u of it; token: input idx = tid of (sequence, input) pairs, max_q per sequence.
  const int mb = a.max_blocks_per_seq, nq = a.max_q;
  const int b_q = tid / nq, j_q = tid - b_q * nq;
  int k_first = 0, ctx_first = 0, pb_first[8], tok_first = 0;
  if (tid < B) {
    k_first = a.spec_len[tid];
    ctx_first = a.ctx_lens[tid];
  }
  auto token = [&](int b, int j) { return j == 0 ? a.last_tok[b] : a.voted[(size_t)b * a.k_max + j - 1]; };  // (j < max_q <= k_max + 1)
  if (blockIdx.x == 0) {
    const long last = (long)B * mb - 1;
#pragma unroll
    for (int u = 0; u < 8; ++u) pb_first[u] = a.block_tables[min((long)(tid + u * PREP_THREADS), last)];
    if (a.last_tok) tok_first = token(min(b_q, B - 1), j_q);
  }
  if (tid == 0) { s_bad = 0; s_tiles = 0ull; }
  __syncthreads();
  // pass 1: per-sequence validation
  for (int b = tid; b < B; b += PREP_THREADS) {
    const int k = b == tid ? k_first : a.spec_len[b];
    const int ctx = b == tid ? ctx_first : a.ctx_lens[b];
    const bool fits = k >= 0 && k <= a.k_max && k < a.max_q;  // (the attention launches were sized for max_q rows)
    s_row0[b + 1] = fits ? k + 1 : 1;
    s_ctx[b] = ctx;
    if (blockIdx.x > 0) continue;
    int ok = 1;
    int flags = 0;
    int nb = 0;
    if (!fits) { ok = 0; flags |= MN_DEV_SPEC_LEN; }
    if (ok) {
      const long need = (long)ctx + k + 1;
      if (ctx < 0 || need > (long)a.max_blocks_per_seq * a.block_size) { ok = 0; flags |= MN_DEV_BLOCK_TABLE; }
      if (ok && need > a.max_pos) { ok = 0; flags |= MN_DEV_TOKEN; }
      // the host sized the attention launch (key tiles per split, block-index staging) for max_ctx keys
      if (ok && need > a.max_ctx) { ok = 0; flags |= MN_DEV_CTX; }
      if (ok) nb = (int)((need + a.block_size - 1) / a.block_size);
    }
    s_ok[b] = ok;
    s_nb[b] = ok ? nb : 0;
    if (flags) {
      if (a.dev_status) atomicOr(a.dev_status, flags);
      if (flags & MN_DEV_SPEC_LEN) atomicOr(&s_bad, 1);
    }
  }
  __syncthreads();
  if (blockIdx.x > 0) {                     // (whole workgroup)
    scan_rows(s_row0, B, s_wave);
    rope_rows(a, s_row0, s_ctx);
    return;
  }
  // pass 1b: every mapped block of every sequence, all threads side by side (a long context has hundreds of table
  // entries; one thread walking them is a chain of dependent loads), eight entries per thread in flight
  {
    const int step_b = PREP_THREADS / mb, step_i = PREP_THREADS % mb;
    int b = tid / mb, i = tid % mb;
    for (bool first = true; b < B; first = false) {
      int pb[8], bb[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        bb[u] = b < B && i < s_nb[b] ? b : -1;
        if (first) pb[u] = pb_first[u];
        else pb[u] = bb[u] >= 0 ? a.block_tables[(size_t)b * mb + i] : 0;
        b += step_b;
        i += step_i;
        if (i >= mb) { i -= mb; ++b; }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (bb[u] >= 0 && (pb[u] < 0 || pb[u] >= a.num_blocks)) {
          atomicAnd(&s_ok[bb[u]], 0);
          if (a.dev_status) atomicOr(a.dev_status, MN_DEV_BLOCK_TABLE);
        }
    }
  }
  // pass 1c: every input token of every sequence that passed the shape checks, likewise
  if (a.last_tok) {
    int b = b_q, j = j_q;
    for (bool first = true; b < B; first = false) {
      if (s_nb[b] != 0 && j < s_row0[b + 1]) {  // (s_row0[b+1] still holds q_b = k_b + 1 here)
        const int tok = first ? tok_first : token(b, j);
        if (tok < 0 || tok >= a.vocab) {
          atomicAnd(&s_ok[b], 0);
          if (a.dev_status) atomicOr(a.dev_status, MN_DEV_TOKEN);
        }
      }
      b += PREP_THREADS / nq;
      j += PREP_THREADS % nq;
      if (j >= nq) { j -= nq; ++b; }
    }
  }
  __syncthreads();
  scan_rows(s_row0, B, s_wave);
  if (tid == 0 && s_row0[B] != a.M) {
    s_bad = 1;
    if (a.dev_status) atomicOr(a.dev_status, MN_DEV_SPEC_LEN);
  }
  __syncthreads();
  // a device spec_len that disagrees with the launch geometry disables the whole batch: every sequence, each with an even share
  // of the rows (at least one, at most the host's longest run), so that the attention kernels write zeros to all of them
  if (s_bad != 0) {
    for (int b = tid; b <= B; b += PREP_THREADS) s_row0[b] = (int)((long)a.M * b / B);
    for (int b = tid; b < B; b += PREP_THREADS) s_ok[b] = 0;
    __syncthreads();
  }
  for (int b = tid; b <= B; b += PREP_THREADS) a.seq_row0[b] = s_row0[b];
  for (int b = tid; b < B; b += PREP_THREADS) {
    const int ok = s_ok[b], ctx = ok ? s_ctx[b] : 0, q = s_row0[b + 1] - s_row0[b];
    a.seq_ctx[b] = ctx;
    a.seq_ok[b] = ok;
    // key tiles of 32, once per group of 128 (query position x head) rows: the work of the sequence in units of
    // one workgroup's tile (integer sum: order-free)
    s_nb[b] = ok ? (ctx + q + 31) >> 5 : 0;
    if (ok) atomicAdd(&s_tiles, (unsigned long long)s_nb[b] * (unsigned long long)((q * max(a.q_per_kv, 1) + 127) >> 7));
  }
  // rows: by (sequence, input) pair where that is not many more than the rows, the first of which have their token already; a search
  // for the row's sequence otherwise (thousands of sequences, one of them long)
  const bool pairs = (long)B * nq <= 2l * a.M + PREP_THREADS;
  auto for_rows = [&](auto f) {             // f(row, sequence, input, first)
    if (pairs) {
      int b = b_q, j = j_q;
      for (bool first = true; b < B; first = false) {
        const int row0 = s_row0[b];
        if (j < s_row0[b + 1] - row0) f(row0 + j, b, j, first);
        b += PREP_THREADS / nq;
        j += PREP_THREADS % nq;
        if (j >= nq) { j -= nq; ++b; }
      }
    } else {
      for (int m = tid; m < a.M; m += PREP_THREADS) {
        const int b = seq_of_row(s_row0, B, m);
        f(m, b, m - s_row0[b], false);
      }
    }
  };
  for_rows([&](int m, int b, int j, bool first) {
    const int ok = s_ok[b], p = ok ? s_ctx[b] + j : -1, blk = p / a.block_size;
    a.row_seq[m] = b;
    a.row_j[m] = j;
    a.row_pos[m] = p;
    // where the row's K/V are written, looked up once per step instead of once per layer and head
    a.row_slot[m] = ok ? a.block_tables[(size_t)b * mb + blk] * a.block_size + p - blk * a.block_size : -1;
    a.row_tok[m] = (ok && a.last_tok) ? (first ? tok_first : token(b, j)) : 0;
  });
  if (!a.plan.items) return;
  __syncthreads();
  // ---- the attention work list: one record of 8 int32 per (sequence, row group, KV split) that has work: {sequence, row
  // group, split, splits of the sequence, first row, rows, enabled, context}.  Sequences are ordered by descending key
  // tiles per workgroup (ties by index), so the longest workgroups start first and the short ones fill the end of
  // the launch; the records of the grid past the last real one get sequence = -1.  Ranking is a comparison of every pair of
  // sequences (B <= 4096, once per step): by a wave per sequence while there are few (its lanes also share the records: three
  // prompts of 250 to 700 tokens 47.4 us for the whole call, 52.5 with a thread each), beyond RANK_WAVES of them by a thread for
  // each, or for each four, which reads every entry once.  The whole of mn_attention, 8 heads of 128, 30 to 80 keys, wave and
  // thread: 128 sequences 28.2 and 26.0 us, 256 47.3 and 41.1, 384 68.2 and 55.9, 512 103 and 70, 1024 255 and 130, 4096 2456
  // and 669; 64 ragged sequences of 256 to 2000 keys 78.2 and 77.5.
  // Balance: a workgroup should take about (all key tiles x KV heads) / (the number of workgroups aimed for) tiles, at
  // least min_tiles (below that the lead-in of a workgroup and the partial sums cost more than the parallelism wins).
  // Long sequences of a ragged batch are then cut into more splits than short ones.
  int tps;
  {  // (every thread for itself)
    const unsigned long long w = (unsigned long long)max(a.plan.target_wgs, 1), all = s_tiles * (unsigned long long)max(a.kv_heads, 1) + w - 1;
    const unsigned long long per = all >> 32 ? all / w : (unsigned long long)((uint32_t)all / (uint32_t)w);
    tps = (int)min(max(per, (unsigned long long)max(a.plan.min_tiles, 1)), (unsigned long long)(1 << 20));
  }
  for (int b = tid; b < B; b += PREP_THREADS) {
    const int q = s_row0[b + 1] - s_row0[b], n_tiles = s_nb[b];
    const int n_rg = (((a.q_per_kv * q + 15) >> 4) + a.plan.tiles16_per_wg - 1) / a.plan.tiles16_per_wg;
    const int spl = max(1, min(a.plan.n_splits_max, (n_tiles + tps - 1) / max(tps, 1)));
    s_spl[b] = spl;
    s_cnt[b] = n_rg * spl;                  // a disabled sequence keeps one workgroup per row group: it writes zeros
    // order of the list in one number: longest workgroups first, then by index
    s_nb[b] = (min((n_tiles + spl - 1) / spl, (1 << 19) - 1) << 12) | (MN_MAX_BATCH - 1 - b);
  }
  __syncthreads();
  for_rows([&](int m, int b, int, bool) { a.plan.row_splits[m] = s_spl[b]; });  // for the merge
  // records of sequence b, at place `off` of the list
  auto write_records = [&](int b, int off, int first, int step) {
    const int cnt = s_cnt[b], spl = s_spl[b];
    const int row0 = s_row0[b], q = s_row0[b + 1] - row0, ok = s_ok[b], ctx = ok ? s_ctx[b] : 0;
    for (int i = first; i < cnt; i += step) {
      if (off + i >= a.plan.grid_items) break;  // (cannot happen: the grid holds every real record)
      int4* rec = reinterpret_cast<int4*>(a.plan.items) + 2 * (size_t)(off + i);
      rec[0] = make_int4(b, i / spl, i % spl, spl);
      rec[1] = make_int4(row0, q, ok, ctx);
    }
  };
  int total = 0;
  auto rank_by_thread = [&](auto n_c) {
    constexpr int N = decltype(n_c)::value;
    int key[N], off[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int b = tid + u * PREP_THREADS;
      key[u] = b < B ? s_nb[b] : 0x7fffffff;
      off[u] = 0;
    }
#pragma unroll 8
    for (int b2 = 0; b2 < B; ++b2) {
      const int c = s_cnt[b2], k2 = s_nb[b2];
      total += c;
#pragma unroll
      for (int u = 0; u < N; ++u) off[u] += k2 > key[u] ? c : 0;
    }
#pragma unroll
    for (int u = 0; u < N; ++u)
      if (tid + u * PREP_THREADS < B) write_records(tid + u * PREP_THREADS, off[u], 0, 1);
  };
  static_assert(MN_MAX_BATCH == 4096 && MN_MAX_BATCH <= 4 * PREP_THREADS, "order and ranking by thread");
  if (B > PREP_THREADS) {
    rank_by_thread(IntC<4>{});
  } else if (B > RANK_WAVES) {
    rank_by_thread(IntC<1>{});
  } else {
    for (int b = tid >> 6; b < B; b += PREP_THREADS / 64) {
      const int lane = tid & 63, key = s_nb[b], c = lane < B ? s_cnt[lane] : 0;  // (at most 64 sequences)
      total = wave_sum_i(c);
      const int off = wave_sum_i(lane < B && s_nb[lane] > key ? c : 0);
      write_records(b, off, lane, 64);
    }
  }
  if ((tid >> 6) < B)                       // (every wave that had a sequence knows the total)
    for (int i = total + tid; i < a.plan.grid_items; i += min(B, PREP_THREADS / 64) * 64)
      reinterpret_cast<int4*>(a.plan.items)[2 * (size_t)i] = make_int4(-1, 0, 0, 1);
}

hipError_t launch_prepare(const PrepArgs& a, hipStream_t st) {
  const size_t smem = (size_t)6 * (a.B + 1) * sizeof(int32_t);
  // once per process, whichever thread comes first; a refusal is returned by every call and nothing is launched
  static std::once_flag attr_once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [] {
    attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(prepare_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)(6 * (MN_MAX_BATCH + 1) * sizeof(int32_t)));
  });
  if (attr_err != hipSuccess) return attr_err;
  const int rows = a.rope_half > 0 ? PREP_THREADS / a.rope_half : 1;
  const int rope_wgs = a.rope_half > 0 && a.M > 0 ? (a.M + rows - 1) / rows : 0;
  prepare_kernel<<<1 + rope_wgs, PREP_THREADS, smem, st>>>(a.spec_len, a.ctx_lens, a.block_tables, a.last_tok, a.voted, a.B, a.max_q, a.max_blocks_per_seq, a.k_max, a);
  return hipSuccess;
}

// ------------------------------------------------------------------------------------------
// norm: x += sum of partials + bias (or x = embedding), then LayerNorm / RMSNorm -> h
// ------------------------------------------------------------------------------------------
// Bound by its chain of round trips (row, partial sums, statistics, output) up to a few hundred rows, by the partial sums'
// bytes beyond.  16 waves per row: the row's partial sums are many independent streams; 4 for rows of up to 1024 elements, where
// the waves' exchange is most of the time (16 rows of 768 in a drafting model: 4.1 -> 3.8 us; 40 rows of 5120: 7.0 -> 6.3).  Gains and shifts are asked for with the
// row, not behind the statistics.
constexpr int NORM_MAX_VEC = 2;     // float4 per thread: d <= 1024*2*4 = 8192

template <typename T>
__device__ __forceinline__ float4 load4(const T* p);
template <>
__device__ __forceinline__ float4 load4<float>(const float* p) { return *reinterpret_cast<const float4*>(p); }
template <>
__device__ __forceinline__ float4 load4<bf16_t>(const bf16_t* p) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                     __uint_as_float(u.y & 0xFFFF0000u));
}
template <>
__device__ __forceinline__ float4 load4<f16_t>(const f16_t* p) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  const f16x2 a = __builtin_bit_cast(f16x2, u.x), b = __builtin_bit_cast(f16x2, u.y);
  return make_float4((float)a[0], (float)a[1], (float)b[0], (float)b[1]);
}
// (fp16 stores saturate and set `bad`, see sat_h)
template <typename T>
__device__ __forceinline__ void store4(T* p, float4 v, bool& bad);
template <>
__device__ __forceinline__ void store4<f16_t>(f16_t* p, float4 v, bool& bad) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack2h_sat(v.x, v.y, bad), pack2h_sat(v.z, v.w, bad));
}
template <>
__device__ __forceinline__ void store4<float>(float* p, float4 v, bool&) { *reinterpret_cast<float4*>(p) = v; }
// one element in the activation type TA / the page storage type T; fp16 saturates to the fp16 range
template <typename T>
__device__ __forceinline__ void store1(T* p, float v, bool& bad) { Store<T>::store(p, v); }
template <>
__device__ __forceinline__ void store1<f16_t>(f16_t* p, float v, bool& bad) { *p = (f16_t)sat_h(v, bad); }

// T: storage type of the embedding tables; TA: activation type of the normalised output
template <typename T, typename TA, int NORM_THREADS>
__global__ void __launch_bounds__(NORM_THREADS) norm_kernel(float* x_, const float* partials_, const float* gain_, const float* shift_,
                                                             const void* tok_emb_, int d_, int M_, int n_partials_, NormArgs a) {
  a.x = x_; a.partials = partials_; a.gain = gain_; a.shift = shift_;  // (launch.h: leading arguments)
  a.tok_emb = tok_emb_; a.d = d_; a.M = M_; a.n_partials = n_partials_;
  __shared__ float red[2][NORM_THREADS / 64];
  const int m = blockIdx.x;
  const int tid = threadIdx.x;
  const int d = a.d;
  const int nvec = d >> 2;
  float4 v[NORM_MAX_VEC], gn[NORM_MAX_VEC], sh[NORM_MAX_VEC];
#pragma unroll
  for (int it = 0; it < NORM_MAX_VEC; ++it) {
    const int e = min(it * NORM_THREADS + tid, nvec - 1) << 2;
    gn[it] = *reinterpret_cast<const float4*>(a.gain + e);
    if (a.shift) sh[it] = *reinterpret_cast<const float4*>(a.shift + e);
  }
  float* xr = a.x + (size_t)m * d;
  const bool embed = a.tok_emb != nullptr;
  const T* te = embed ? reinterpret_cast<const T*>(a.tok_emb) + (size_t)a.row_tok[m] * d : nullptr;
  const int pos = (embed && a.pos_emb) ? (a.row_pos[m] < 0 ? 0 : a.row_pos[m]) : 0;
  const T* pe = (embed && a.pos_emb) ? reinterpret_cast<const T*>(a.pos_emb) + (size_t)pos * d : nullptr;
  float sum = 0.f;
#pragma unroll
  for (int it = 0; it < NORM_MAX_VEC; ++it) {
    const int i4 = it * NORM_THREADS + tid;
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i4 < nvec) {
      const int e = i4 << 2;
      if (embed) {
        r = load4<T>(te + e);
        if (pe) {
          const float4 p = load4<T>(pe + e);
          r.x += p.x; r.y += p.y; r.z += p.z; r.w += p.w;
        }
      } else {
        r = *reinterpret_cast<const float4*>(xr + e);
        if (a.partials) {
          // fixed summation order: residual, then partial 0, 1, ..., then the bias.  The partials are
          // fetched eight at a time before any is added (indices past the end repeat the last one and are
          // not added): one memory round trip per batch instead of one per partial
          for (int s0 = 0; s0 < a.n_partials; s0 += 8) {
            float4 p[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
              p[j] = *reinterpret_cast<const float4*>(a.partials + ((size_t)min(s0 + j, a.n_partials - 1) * a.M + m) * d + e);
#pragma unroll
            for (int j = 0; j < 8; ++j)
              if (s0 + j < a.n_partials) { r.x += p[j].x; r.y += p[j].y; r.z += p[j].z; r.w += p[j].w; }
          }
        }
        if (a.bias) {
          const float4 p = *reinterpret_cast<const float4*>(a.bias + e);
          r.x += p.x; r.y += p.y; r.z += p.z; r.w += p.w;
        }
      }
      if (embed || a.partials || a.bias) *reinterpret_cast<float4*>(xr + e) = r;
      sum += (r.x + r.y) + (r.z + r.w);
    }
    v[it] = r;
  }
  const float inv_d = 1.f / (float)d;
  float mean = 0.f;
  if (a.shift) mean = block_sum<NORM_THREADS / 64, true>(sum, red[0]) * inv_d;
  float sq = 0.f;
#pragma unroll
  for (int it = 0; it < NORM_MAX_VEC; ++it) {
    const int i4 = it * NORM_THREADS + tid;
    if (i4 < nvec) {
      const float4 r = v[it];
      const float a0 = r.x - mean, a1 = r.y - mean, a2 = r.z - mean, a3 = r.w - mean;
      sq += (a0 * a0 + a1 * a1) + (a2 * a2 + a3 * a3);
    }
  }
  const float var = block_sum<NORM_THREADS / 64, true>(sq, red[1]) * inv_d;
  const float rstd = 1.f / sqrtf(var + a.eps);
  if (a.rstd && tid == 0) a.rstd[m] = rstd;
  TA* hr = reinterpret_cast<TA*>(a.h) + (size_t)m * d;
  bool bad = false;
#pragma unroll
  for (int it = 0; it < NORM_MAX_VEC; ++it) {
    const int i4 = it * NORM_THREADS + tid;
    if (i4 < nvec) {
      const int e = i4 << 2;
      const float4 r = v[it];
      const float4 g = gn[it];
      float4 o = make_float4((r.x - mean) * rstd * g.x, (r.y - mean) * rstd * g.y, (r.z - mean) * rstd * g.z,
                             (r.w - mean) * rstd * g.w);
      if (a.shift) {
        o.x += sh[it].x; o.y += sh[it].y; o.z += sh[it].z; o.w += sh[it].w;
      }
      store4<TA>(a.operand ? reinterpret_cast<TA*>(a.h) + operand_at(m, e, a.M, d) : hr + e, o, bad);
    }
  }
  if (bad && a.dev_status) atomicOr(a.dev_status, MN_DEV_RANGE);
}

void launch_norm(const NormArgs& a, hipStream_t st) {
  if (a.M <= 0) return;
  const bool narrow = a.d <= 1024;
  auto launch = [&](auto kernel, int threads) {
    kernel<<<a.M, threads, 0, st>>>(a.x, a.partials, a.gain, a.shift, a.tok_emb, a.d, a.M, a.n_partials, a);
  };
  if (a.dtype == MN_DT_BF16) narrow ? launch(norm_kernel<bf16_t, f16_t, 256>, 256) : launch(norm_kernel<bf16_t, f16_t, 1024>, 1024);
  else narrow ? launch(norm_kernel<float, float, 256>, 256) : launch(norm_kernel<float, float, 1024>, 1024);
}

// ------------------------------------------------------------------------------------------
// rotary embedding + tentative KV append
// ------------------------------------------------------------------------------------------
// grid (ceil(heads / heads per block), M), 256 threads: a thread owns W pairs (t .. t+W-1, and + hd/2) of one head, so a
// block takes 512 W / hd consecutive heads of one row.  Four (16-byte loads of the partial sums) where most heads are query heads,
// whose four elements are stored at once, and there are many rows: the elements of a K/V row go to the pages one by one, and
// those stores are slower the fewer threads share them.  Four and one pair: 64 query heads of 128 over 8 KV heads 22.6 and 28.3 us
// at 844 rows, 14.5 and 16.2 at 400, 11.4 both at 256, 7.9 both at 144 (a four-layer step 1590 and 1596), 6.5 and 6.0 at 96 (1452
// and 1451); 32 over 8 22.7 and 29.4 at 1500 rows; 32 over 16 24.1 and 16.0 at 520; 40 over 40 67.3 and 42.0 at 844, 16.4 and 11.0
// at 144.
// TA: activation type of the query buffer; T: storage type of the KV pages
constexpr int ROPE_THREADS = 256;
constexpr int ROPE_WIDE_ROWS = 97, ROPE_WIDE_GROUP = 4;  // fewest rows and query heads per KV head for four pairs
template <typename TA, typename T, int W>
__global__ void __launch_bounds__(ROPE_THREADS) rope_append_kernel(const int32_t* row_slot_, const float* qkv_, const float* rope_cos_,
                                                                    const float* rope_sin_, int H_, int Hkv_, int hd_, int n_partials_,
                                                                    int M_, RopeAppendArgs a) {
  a.rows.row_slot = row_slot_; a.qkv = qkv_; a.rope_cos = rope_cos_; a.rope_sin = rope_sin_;  // (launch.h: leading arguments)
  a.H = H_; a.Hkv = Hkv_; a.hd = hd_; a.n_partials = n_partials_; a.M = M_;
  struct alignas(4 * W) Piece { float x[W]; };
  struct alignas(4) PieceU { float x[W]; };                    // (biases start at any float's address)
  constexpr int PB = W == 1 ? 8 : 4;                           // partial sums in flight
  const int m = blockIdx.y;
  const int hd = a.hd, half = hd >> 1, qw = half / W;          // (head_dim is a multiple of 8)
  const int head = blockIdx.x * (ROPE_THREADS / qw) + (int)threadIdx.x / qw;
  const int t = ((int)threadIdx.x % qw) * W;
  if (head >= a.H + 2 * a.Hkv) return;
  const int slot = a.rows.row_slot[m];  // (asked for first: the stores at the end wait for nothing else)
  const int ncols = (a.H + 2 * a.Hkv) * hd;
  const int c0 = head * hd + t, c1 = c0 + half;
  const bool is_v = head >= a.H + a.Hkv, turn = a.rope_cos && !is_v;
  Piece cs, sn, v0, v1;
#pragma unroll
  for (int e = 0; e < W; ++e) { cs.x[e] = 1.f; sn.x[e] = v0.x[e] = v1.x[e] = 0.f; }
  if (turn) {
    cs = *reinterpret_cast<const Piece*>(a.rope_cos + (size_t)m * half + t);
    sn = *reinterpret_cast<const Piece*>(a.rope_sin + (size_t)m * half + t);
  }
  // partials fetched PB at a time before any is added (see norm_kernel); the order of the sum is fixed
  for (int s0 = 0; s0 < a.n_partials; s0 += PB) {
    Piece p0[PB], p1[PB];
#pragma unroll
    for (int j = 0; j < PB; ++j) {
      const float* p = a.qkv + ((size_t)min(s0 + j, a.n_partials - 1) * a.M + m) * ncols;
      p0[j] = *reinterpret_cast<const Piece*>(p + c0);
      p1[j] = *reinterpret_cast<const Piece*>(p + c1);
    }
#pragma unroll
    for (int j = 0; j < PB; ++j)
      if (s0 + j < a.n_partials) {
#pragma unroll
        for (int e = 0; e < W; ++e) { v0.x[e] += p0[j].x[e]; v1.x[e] += p1[j].x[e]; }
      }
  }
  if (a.bias) {
    const PieceU b0 = *reinterpret_cast<const PieceU*>(a.bias + c0), b1 = *reinterpret_cast<const PieceU*>(a.bias + c1);
#pragma unroll
    for (int e = 0; e < W; ++e) { v0.x[e] += b0.x[e]; v1.x[e] += b1.x[e]; }
  }
  if (turn) {
#pragma unroll
    for (int e = 0; e < W; ++e) {
      const float x = v0.x[e], y = v1.x[e];
      v0.x[e] = x * cs.x[e] - y * sn.x[e];
      v1.x[e] = y * cs.x[e] + x * sn.x[e];
    }
  }
  bool bad = false;
  if (head < a.H) {
    TA* q = reinterpret_cast<TA*>(a.q) + ((size_t)m * a.H + head) * hd;
    if constexpr (W == 4) {
      store4<TA>(q + t, make_float4(v0.x[0], v0.x[1], v0.x[2], v0.x[3]), bad);
      store4<TA>(q + t + half, make_float4(v1.x[0], v1.x[1], v1.x[2], v1.x[3]), bad);
    } else {
      store1<TA>(q + t, v0.x[0], bad);
      store1<TA>(q + t + half, v1.x[0], bad);
    }
    if (bad && a.dev_status) atomicOr(a.dev_status, MN_DEV_RANGE);
    return;
  }
  if (slot < 0) return;  // disabled sequence: nothing is written to the cache (and nothing reported)
  const int bs = a.kv.block_size;
  const int pb = slot / bs;
  const int off = slot % bs;
  if (!is_v) {
    const int kh = head - a.H;
    T* base = reinterpret_cast<T*>(a.kv.k) + ((size_t)pb * a.Hkv + kh) * (size_t)hd * bs;
    // [hd/8][bs][8]: the W elements are neighbours inside their piece of eight
    T* k0 = base + ((size_t)(t >> 3) * bs + off) * 8 + (t & 7);
    T* k1 = base + ((size_t)((t + half) >> 3) * bs + off) * 8 + ((t + half) & 7);
#pragma unroll
    for (int e = 0; e < W; ++e) {
      store1<T>(k0 + e, v0.x[e], bad);
      store1<T>(k1 + e, v1.x[e], bad);
    }
  } else {
    const int vh = head - a.H - a.Hkv;
    T* base = reinterpret_cast<T*>(a.kv.v) + ((size_t)pb * a.Hkv + vh) * (size_t)hd * bs;
    // [hd][bs]
#pragma unroll
    for (int e = 0; e < W; ++e) {
      store1<T>(base + (size_t)(t + e) * bs + off, v0.x[e], bad);
      store1<T>(base + (size_t)(t + half + e) * bs + off, v1.x[e], bad);
    }
  }
  if (bad && a.dev_status) atomicOr(a.dev_status, MN_DEV_RANGE);
}

template <int W>
static void launch_rope_w(const RopeAppendArgs& a, hipStream_t st) {
  const int per_block = ROPE_THREADS / (a.hd / (2 * W));  // head_dim is one of 8 ... 256: hd/8 divides 256
  dim3 grid((a.H + 2 * a.Hkv + per_block - 1) / per_block, a.M);
  auto launch = [&](auto kernel) {
    kernel<<<grid, ROPE_THREADS, 0, st>>>(a.rows.row_slot, a.qkv, a.rope_cos, a.rope_sin, a.H, a.Hkv, a.hd, a.n_partials, a.M, a);
  };
  a.dtype == MN_DT_BF16 ? launch(rope_append_kernel<f16_t, f16_t, W>) : launch(rope_append_kernel<float, float, W>);
}
void launch_rope_append(const RopeAppendArgs& a, hipStream_t st) {
  if (a.M <= 0) return;
  if (a.M >= ROPE_WIDE_ROWS && a.H >= ROPE_WIDE_GROUP * a.Hkv) launch_rope_w<4>(a, st);
  else launch_rope_w<1>(a, st);
}

// ------------------------------------------------------------------------------------------
// FFN activation on the first projection's partial sums
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ void __launch_bounds__(256) act_kernel(ActArgs a) {
  const size_t nvec = (size_t)a.M * (a.F >> 2);
  const int ncols = a.swiglu ? 2 * a.F : a.F;
  bool bad = false;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += (size_t)gridDim.x * blockDim.x) {
    const int m = (int)(i / (a.F >> 2));
    const int f = (int)(i % (a.F >> 2)) << 2;
    float4 g = make_float4(0.f, 0.f, 0.f, 0.f), u = g;
    for (int s = 0; s < a.n_partials; ++s) {
      const float* p = a.partials + ((size_t)s * a.M + m) * ncols;
      const float4 x = *reinterpret_cast<const float4*>(p + f);
      g.x += x.x; g.y += x.y; g.z += x.z; g.w += x.w;
      if (a.swiglu) {
        const float4 y = *reinterpret_cast<const float4*>(p + a.F + f);
        u.x += y.x; u.y += y.y; u.z += y.z; u.w += y.w;
      }
    }
    float4 o;
    if (a.swiglu) {
      o.x = g.x / (1.f + __expf(-g.x)) * u.x;
      o.y = g.y / (1.f + __expf(-g.y)) * u.y;
      o.z = g.z / (1.f + __expf(-g.z)) * u.z;
      o.w = g.w / (1.f + __expf(-g.w)) * u.w;
    } else {
      if (a.bias) {
        const float4 bb = *reinterpret_cast<const float4*>(a.bias + f);
        g.x += bb.x; g.y += bb.y; g.z += bb.z; g.w += bb.w;
      }
      o = make_float4(fmaxf(g.x, 0.f), fmaxf(g.y, 0.f), fmaxf(g.z, 0.f), fmaxf(g.w, 0.f));
    }
    store4<T>(reinterpret_cast<T*>(a.act) + (size_t)m * a.F + f, o, bad);
  }
  if (bad && a.dev_status) atomicOr(a.dev_status, MN_DEV_RANGE);
}

void launch_act(const ActArgs& a, hipStream_t st) {
  if (a.M <= 0) return;
  const size_t nvec = (size_t)a.M * (a.F >> 2);
  int blocks = (int)((nvec + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  if (a.dtype == MN_DT_BF16) act_kernel<f16_t><<<blocks, 256, 0, st>>>(a);
  else act_kernel<float><<<blocks, 256, 0, st>>>(a);
}

// ------------------------------------------------------------------------------------------
// vocabulary argmax: lowest id attaining the row maximum; NaN never wins
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void arg_better(float& bv, int& bi, float v, int i) {
  if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
}

// One workgroup per row with eight 16-byte pieces in flight per thread.  Up to ARGMAX_WIDE_ROWS rows (fewer than CUs) it has 16
// waves: a row of 32000 scores is asked for at once (16 rows 9.6 -> 7.3 us, 6.5 since the row's place is asked for with the scores and
// one wave compares the waves' results); with more rows the chip is full either way and
// 4 waves leave more workgroups per CU (618 rows 17.8 us, 25.0 with 16 waves).  It also adds up the partial sums of a
// split vocabulary projection (144 rows of 32000 scores in two splits, when that head was still split: 22 us as a launch of its own and the
// argmax, 14 together).
constexpr int ARGMAX_WIDE_ROWS = 256;
template <int ARGMAX_THREADS>
__global__ void __launch_bounds__(ARGMAX_THREADS) argmax_rows_kernel(float* __restrict__ logits, const float* __restrict__ partials,
                                                                     int S, int M, int V, RowInfo rows, int k_max,
                                                                     int32_t* __restrict__ greedy, int B) {
  constexpr int NW = ARGMAX_THREADS / 64;
  __shared__ float sv[NW];
  __shared__ int si[NW];
  const int tid = threadIdx.x;
  if ((int)blockIdx.x >= M) {
    // padding blocks: one per sequence
    const int b = blockIdx.x - M;
    const int q = rows.seq_ok[b] ? rows.seq_row0[b + 1] - rows.seq_row0[b] : 0;
    for (int j = q + tid; j <= k_max; j += blockDim.x) greedy[(size_t)b * (k_max + 1) + j] = -1;
    return;
  }
  const int m = blockIdx.x;
  const int b = rows.row_seq[m], row_j = rows.row_j[m], ok = rows.seq_ok[b];  // (asked for first: the answer waits for nothing else)
  float* r = logits + (size_t)m * V;
  const float* src = partials ? partials + (size_t)m * V : r;
  const size_t stride = (size_t)M * V;
  float bv = -INFINITY;
  int bi = 0x7FFFFFFF;
  if ((V & 3) == 0 && (reinterpret_cast<uintptr_t>(logits) & 15) == 0) {
    // 16-byte pieces, eight in flight per thread before any is looked at (one piece per round trip is bound
    // by memory latency); a thread's indices grow, and ties between threads are settled by arg_better
    const int n4 = V >> 2;
    for (int i0 = tid; i0 < n4; i0 += 8 * ARGMAX_THREADS) {
      float4 p[8];
      if (i0 - tid + ARGMAX_THREADS >= n4) {  // (uniform: short rows have one piece per thread)
        p[0] = reinterpret_cast<const float4*>(src)[min(i0, n4 - 1)];
#pragma unroll
        for (int u = 1; u < 8; ++u) p[u] = p[0];
      } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = reinterpret_cast<const float4*>(src)[min(i0 + u * ARGMAX_THREADS, n4 - 1)];
      }
      if (partials) {
        for (int s = 1; s < S; ++s) {       // (fixed order)
          float4 x[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) x[u] = reinterpret_cast<const float4*>(src + s * stride)[min(i0 + u * ARGMAX_THREADS, n4 - 1)];
#pragma unroll
          for (int u = 0; u < 8; ++u) { p[u].x += x[u].x; p[u].y += x[u].y; p[u].z += x[u].z; p[u].w += x[u].w; }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (i0 + u * ARGMAX_THREADS < n4) reinterpret_cast<float4*>(r)[i0 + u * ARGMAX_THREADS] = p[u];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i4 = i0 + u * ARGMAX_THREADS;
        if (i4 < n4) {
          arg_better(bv, bi, p[u].x, 4 * i4);
          arg_better(bv, bi, p[u].y, 4 * i4 + 1);
          arg_better(bv, bi, p[u].z, 4 * i4 + 2);
          arg_better(bv, bi, p[u].w, 4 * i4 + 3);
        }
      }
    }
  } else {
    for (int i = tid; i < V; i += ARGMAX_THREADS) {
      float v = src[i];
      if (partials) {
        for (int s = 1; s < S; ++s) v += src[s * stride + i];
        r[i] = v;
      }
      arg_better(bv, bi, v, i);
    }
  }
  auto meet = [&](uint32_t v, uint32_t i) { arg_better(bv, bi, __uint_as_float(v), (int)i); };
  auto row_of_16 = [&](bool all) {                           // (all: 16 lanes, else 4)
    meet(lane_swap<LANE_1>(__float_as_uint(bv)), lane_swap<LANE_1>((uint32_t)bi));
    meet(lane_swap<LANE_2>(__float_as_uint(bv)), lane_swap<LANE_2>((uint32_t)bi));
    if (!all) return;
    meet(lane_swap<LANE_4>(__float_as_uint(bv)), lane_swap<LANE_4>((uint32_t)bi));
    meet(lane_swap<LANE_8>(__float_as_uint(bv)), lane_swap<LANE_8>((uint32_t)bi));
  };
  auto across = [&](auto dist) {
    uint32_t va, vb, ia, ib;
    lane_pair<decltype(dist)::value>(__float_as_uint(bv), va, vb);
    lane_pair<decltype(dist)::value>((uint32_t)bi, ia, ib);
    bv = __uint_as_float(va);
    bi = (int)ia;
    meet(vb, ib);
  };
  row_of_16(true);
  across(IntC<16>{});
  across(IntC<32>{});
  if ((tid & 63) == 0) { sv[tid >> 6] = bv; si[tid >> 6] = bi; }
  __syncthreads();
  if (tid < 64) {
    bv = sv[min(tid, NW - 1)];
    bi = si[min(tid, NW - 1)];
    static_assert(NW == 16 || NW == 4, "the waves' results in one row of lanes");
    row_of_16(NW == 16);
    if (bi >= V) bi = 0;
    if (tid == 0 && ok) greedy[(size_t)b * (k_max + 1) + row_j] = bi;
  }
}

void launch_argmax_rows(float* logits, const float* partials, int S, int M, int V, const RowInfo& rows, int k_max,
                        int32_t* greedy, int B, hipStream_t st) {
  if (M + B <= 0) return;
  if (M <= ARGMAX_WIDE_ROWS) argmax_rows_kernel<1024><<<M + B, 1024, 0, st>>>(logits, partials, S, M, V, rows, k_max, greedy, B);
  else argmax_rows_kernel<256><<<M + B, 256, 0, st>>>(logits, partials, S, M, V, rows, k_max, greedy, B);
}

}  // namespace mn
