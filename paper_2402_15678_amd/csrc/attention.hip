// Multi-token paged attention against an existing KV cache (paper section 4: paged attention
// extended to more than one input token per sequence once a cache exists).  Query row j of
// sequence b sees the cached keys [0, ctx_b) and the new keys 0..j of its own sequence.
//
// The keys and values of the scored tokens themselves are in the pages already: the tentative append
// (rope_append_kernel) runs before attention, so the kernels here read nothing but pages.
//
// Three kernels:
//  * attn_mfma_kernel  fp16 pages / fp16 queries, head_dim 128, 16-token blocks.  The G*q_b query rows that share one
//    KV head (grouped-query attention stacks the group's heads on top of the speculated tokens)
//    are the column index of every MFMA, so each K/V byte is read once per KV head.  Key tiles go
//    HBM -> LDS by direct loads, already in the operand order of the MFMAs of all the
//    waves: the page layouts put 8 consecutive contraction elements in 16 bytes for both
//    products (head-dim chunks for K, tokens for V).  The KV range of a sequence is split across
//    workgroups; partial (max, sum, output) triples are merged by attn_merge_kernel.
//  * attn_keys_kernel  fp16 pages / fp16 queries, head_dim 64 or 128, 16-token blocks, few stacked query rows per KV head
//    (decoding token by token, models without head groups, drafting models): the waves split the keys.
//  * attn_generic_kernel  any storage type / head_dim / block size; plain FMA, one (row, head)
//    per workgroup.  Used by the fp32 model and as the fallback.
#include "launch.h"
#include "tune.h"
#include "../../include/minions_verify.h"

#include <mutex>

namespace mn {

// ------------------------------------------------------------------------------------------
// generic kernel
// ------------------------------------------------------------------------------------------
// 256 threads; 1024 beyond 256 keys of context where every workgroup has a CU to itself, and up to two per CU at contexts beyond
// 1024 keys: a chunk of keys is one round trip to the pages and back, whatever its size.  With more workgroups the round trips
// of one hide behind another's, and 1024 threads only leave fewer of them on a CU, most of their threads idle on a prompt's early
// rows.  Measured with cold pages (head_dim 32 to 256, fp32 and fp16 pages, 1 to 1000 rows, even and ragged contexts), 1024
// against 256 threads: up to 256 workgroups 0.67 to 1.01 of the time; 257 to 512 workgroups 0.88 to 1.16 at 300 and 700 keys, 0.80
// to 1.12 (0.97 on average) at 1500, 0.60 to 1.05 (0.91) at 3000 and 6000; 513 to 1024 workgroups 0.81 to 1.37 (1.12); beyond 4096
// 1.05 to 2.30 (a drafting model's 16 prompts of 300 tokens 1073 us with 256, 1740 with 1024).
constexpr int GEN_ALONE = 256, GEN_PAIRS = 512, GEN_LONG = 1024;

// TA: activation type of q and out; T: storage type of the KV pages
// FUSED (fp32 models, few rows per sequence): the workgroup adds up its query and the K and V rows of this step that the query
// sees from the QKV sums itself (in dynamic LDS, GEN_NEW_ROWS at most) and reads only older keys from the pages, to which the first
// head of a KV head's group writes the row's own: no rotary/append launch.  Bound by its chain (row, block ids, keys, softmax,
// values, and before them the QKV sums): 5 rows x 4 heads of 64 over 69 keys 7.5 us and 3.1 for the append before, 5.3 with the keys'
// pieces and the first values asked for at once, 6.7 with the append inside.
constexpr int GEN_NEW_ROWS = 17;
constexpr int GEN_KPIECES = 8;
constexpr int GEN_VPRE = 4;   // groups of four values of a chunk asked for before its softmax
template <typename TA, typename T, int GEN_THREADS, bool FUSED>
__global__ void __launch_bounds__(GEN_THREADS) attn_generic_kernel(const int32_t* row_seq_, const int32_t* row_pos_, const int32_t* row_j_,
                                                                    const int32_t* row_slot_, const int32_t* block_tables_, int H_,
                                                                    int Hkv_, int hd_, int block_size_, AttnArgs a) {
  a.rows.row_seq = row_seq_; a.rows.row_pos = row_pos_; a.rows.row_j = row_j_; a.rows.row_slot = row_slot_;  // (launch.h: leading
  a.kv.block_tables = block_tables_; a.H = H_; a.Hkv = Hkv_; a.hd = hd_; a.kv.block_size = block_size_;      // arguments)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* s_new = reinterpret_cast<float*>(smem);  // [2][rows of the sequence up to m][hd]: K, V
  __shared__ float s_q[256];
  __shared__ __attribute__((aligned(16))) float s_p[GEN_THREADS];
  __shared__ uint64_t s_at[GEN_THREADS];  // element 0 of a key's V column in the pages (element i: + i * bs), found once per chunk
  __shared__ float s_red[GEN_THREADS / 64];
  __shared__ float s_acc[GEN_THREADS];
  const int h = blockIdx.x, m = blockIdx.y, tid = threadIdx.x;
  const int hd = a.hd, bs = a.kv.block_size;
  const int b = a.rows.row_seq[m];
  const int pos = a.rows.row_pos[m];
  TA* o = reinterpret_cast<TA*>(a.out) + ((size_t)m * a.H + h) * hd;
  if (pos < 0) {
    for (int e = tid; e < hd; e += GEN_THREADS) Store<TA>::store(o + e, 0.f);
    return;
  }
  const int nkeys = pos + 1;
  const int kh = h / (a.H / a.Hkv);
  const float scale = rsqrtf((float)hd);
  const T* Kp = reinterpret_cast<const T*>(a.kv.k);
  const T* Vp = reinterpret_cast<const T*>(a.kv.v);
  const int32_t* bt = a.kv.block_tables + (size_t)b * a.kv.max_blocks_per_seq;
  int old = nkeys;                  // keys read from the pages
  if constexpr (FUSED) {
    const int j = a.rows.row_j[m], slot = a.rows.row_slot[m], half = hd >> 1, ncols = (a.H + 2 * a.Hkv) * hd;
    old = pos - j;
    // item = one pair (t, t + hd/2): of the query, then of the K rows, then of the V rows
    for (int idx = tid; idx < (2 * j + 3) * half; idx += GEN_THREADS) {
      const int t = idx & (half - 1), which = idx >> (31 - __clz(half));          // 0: query; 1 .. j + 1: K of row which - 1; then V
      const bool is_q = which == 0, is_v = which > j + 1;
      const int jj = is_q ? j : (is_v ? which - j - 2 : which - 1), mm = m - j + jj;
      const int c = (is_q ? h : (is_v ? a.H + a.Hkv : a.H) + kh) * hd + t;
      const float* p = a.qkv + (size_t)mm * ncols + c;
      float x = p[0], y = p[half], bx = 0.f, by = 0.f;
      if (a.bias) { bx = a.bias[c]; by = a.bias[c + half]; }
      for (int s = 1; s < a.n_partials; ++s) {
        x += p[(size_t)s * a.M * ncols];
        y += p[(size_t)s * a.M * ncols + half];
      }
      if (a.bias) { x += bx; y += by; }
      if (a.rope_cos && !is_v) {
        const float cs = a.rope_cos[(size_t)mm * half + t], sn = a.rope_sin[(size_t)mm * half + t], x0 = x;
        x = x0 * cs - y * sn;
        y = y * cs + x0 * sn;
      }
      if (is_q) {
        s_q[t] = x * scale;
        s_q[t + half] = y * scale;
        continue;
      }
      float* r = s_new + ((is_v ? j + 1 : 0) + jj) * hd + t;
      r[0] = x;
      r[half] = y;
      if (jj == j && h % (a.H / a.Hkv) == 0 && slot >= 0) {  // this row's own, to the pages
        T* base = reinterpret_cast<T*>(is_v ? a.kv.v : a.kv.k) + ((size_t)(slot / bs) * a.Hkv + kh) * (size_t)hd * bs;
        const int off = slot % bs, t1 = t + half;
        Store<T>::store(base + (is_v ? (size_t)t * bs + off : ((size_t)(t >> 3) * bs + off) * 8 + (t & 7)), x);
        Store<T>::store(base + (is_v ? (size_t)t1 * bs + off : ((size_t)(t1 >> 3) * bs + off) * 8 + (t1 & 7)), y);
      }
    }
  } else {
    const TA* q = reinterpret_cast<const TA*>(a.q) + ((size_t)m * a.H + h) * hd;
    for (int e = tid; e < hd; e += GEN_THREADS) s_q[e] = Store<TA>::load(q + e) * scale;
  }
  __syncthreads();
  const int ng = GEN_THREADS / hd;  // key groups in the PV phase
  const int e_own = tid & (hd - 1), kg = tid >> (31 - __clz(hd));  // (head_dim is a power of two)
  float run_m = -INFINITY, run_l = 0.f, acc = 0.f;
  for (int k0 = 0; k0 < nkeys; k0 += GEN_THREADS) {
    const int key = k0 + tid;
    float s = -INFINITY;
    const int blk = (int)((uint32_t)key / (uint32_t)bs), off = key - blk * bs;  // (as signed numbers two registers more: the fp32 kernel spilled them)
    uint64_t page = 0;
    if (key < old) {
      page = ((uint64_t)(uint32_t)bt[blk] * a.Hkv + kh) * (uint64_t)(hd * bs);
      s_at[tid] = page + off;
    }
    if (FUSED && key >= old && key < nkeys) {
      const float* kr = s_new + (key - old) * hd;
      float d = 0.f;
      for (int e = 0; e < hd; ++e) d = fmaf(s_q[e], kr[e], d);
      s = d;
    } else if (key < nkeys) {
      float d = 0.f;
      const T* kb = Kp + page;
      // (eight consecutive elements at once, GEN_KPIECES pieces asked for before any is used: left to itself the compiler makes
      // a round trip of every piece)
      struct __attribute__((aligned(sizeof(T)))) Piece { T x[8]; };
      // (heads of 8 elements have one piece, and short contexts one value group per thread: with the repeats of both 4 prompts of 201
      // tokens x 16 fp32 heads of 8 took 48.1 us instead of 39.8, 200 x 41 keys 20.6 instead of 18.1)
      if (hd == 8) {                         // (uniform)
        const Piece k1 = *reinterpret_cast<const Piece*>(kb + (size_t)off * 8);
#pragma unroll
        for (int i = 0; i < 8; ++i) d = fmaf(s_q[i], (float)k1.x[i], d);
      }
      for (int c0 = 0; c0 < hd / 8 && hd > 8; c0 += GEN_KPIECES) {
        Piece kk[GEN_KPIECES];
#pragma unroll
        for (int c = 0; c < GEN_KPIECES; ++c) kk[c] = *reinterpret_cast<const Piece*>(kb + ((size_t)min(c0 + c, hd / 8 - 1) * bs + off) * 8);
        asm volatile("" ::: "memory");
#pragma unroll
        for (int c = 0; c < GEN_KPIECES; ++c) {
          if (c0 + c >= hd / 8) break;       // (uniform)
#pragma unroll
          for (int i = 0; i < 8; ++i) d = fmaf(s_q[(c0 + c) * 8 + i], (float)kk[c].x[i], d);
        }
      }
      s = d;
    }
    // chunk maximum
    float cm = wave_max(s);
    __syncthreads();
    const int cnt = min(GEN_THREADS, nkeys - k0), cnt_old = min(cnt, old - k0);
    // the first values, on their way while the probabilities are worked out: four keys of a block at once (uniform)
    struct __attribute__((aligned(sizeof(T)))) Quad { T x[4]; };
    const int quads = (bs & 3) == 0 ? (cnt_old + 3) >> 2 : 0;
    Quad vpre[GEN_VPRE];
    if (quads > 0) {                  // (repeats past the end are not used)
      vpre[0] = *reinterpret_cast<const Quad*>(Vp + (s_at[4 * min(kg, quads - 1)] + (uint32_t)(e_own * bs)));
      if (quads > ng) {
#pragma unroll
        for (int u = 1; u < GEN_VPRE; ++u) vpre[u] = *reinterpret_cast<const Quad*>(Vp + (s_at[4 * min(kg + u * ng, quads - 1)] + (uint32_t)(e_own * bs)));
      }
    }
    if ((tid & 63) == 0) s_red[tid >> 6] = cm;
    __syncthreads();
    cm = s_red[0];
#pragma unroll
    for (int w = 1; w < GEN_THREADS / 64; ++w) cm = fmaxf(cm, s_red[w]);
    const float new_m = fmaxf(run_m, cm);  // finite: key k0 is always visible
    const float alpha = __expf(run_m - new_m);
    const float p = (key < nkeys) ? __expf(s - new_m) : 0.f;
    s_p[tid] = p;
    const float ps = block_sum<GEN_THREADS / 64>(p, s_red);  // also orders the s_p writes
    run_l = run_l * alpha + ps;
    run_m = new_m;
    acc *= alpha;
    {
      auto add = [&](const Quad& v, int q) {                 // (slots past the last key, and repeats of the last four, may hold anything)
        const f32x4 p4 = *reinterpret_cast<const f32x4*>(s_p + 4 * min(q, GEN_THREADS / 4 - 1));
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in = 4 * q + e < cnt_old;
          acc = fmaf(in ? p4[e] : 0.f, in ? (float)v.x[e] : 0.f, acc);
        }
      };
      if (quads > 0) {
        add(vpre[0], kg);
        if (quads > ng) {
#pragma unroll
          for (int u = 1; u < GEN_VPRE; ++u) add(vpre[u], kg + u * ng);
        }
      }
#pragma unroll 1
      for (int q0 = kg + GEN_VPRE * ng; q0 < quads; q0 += 4 * ng) {
        Quad v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const Quad*>(Vp + (s_at[4 * min(q0 + u * ng, quads - 1)] + (uint32_t)(e_own * bs)));
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < 4; ++u) add(v[u], q0 + u * ng);
      }
      if ((bs & 3) != 0) {
#pragma unroll 8
        for (int i = kg; i < cnt_old; i += ng) acc = fmaf(s_p[i], Store<T>::load(Vp + (s_at[i] + (uint32_t)(e_own * bs))), acc);
      }
      if (FUSED)
        for (int i = max(cnt_old, 0) + kg; i < cnt; i += ng) acc = fmaf(s_p[i], s_new[(pos - old + 1 + k0 + i - old) * hd + e_own], acc);
    }
    __syncthreads();
  }
  s_acc[tid] = (kg < ng) ? acc : 0.f;
  __syncthreads();
  if (tid < hd) {
    float t = 0.f;
    for (int g2 = 0; g2 < ng; ++g2) t += s_acc[g2 * hd + tid];
    Store<TA>::store(o + tid, t / run_l);
  }
}

// ------------------------------------------------------------------------------------------
// MFMA kernel (fp16 pages, fp16 queries, head_dim 128, block 16)
// ------------------------------------------------------------------------------------------
// Workgroup (4 waves) = one (KV head, sequence, row group, KV split).  The R = G*q_b query rows that share the
// KV head are cut into 16-row column tiles; wave w owns tiles w, w+4, (w+8) and keeps their query
// fragments (pre-multiplied by log2(e)/sqrt(hd)) in registers.
//
// Both products have the query row as the MFMA column index (S^T = K Q^T, O^T = V^T P^T): softmax
// statistics are per-lane scalars.  Inside a tile the K rows are permuted (S^T row 4g'+r of half t
// is key 8g' + 4t + r) so that the lane group g of the first product's output holds keys
// 8g..8g+7, exactly the operand order of the second product and 16 contiguous bytes of a V page.
//
// Data path of a key tile (32 keys = two blocks, 16 KB): HBM -> LDS by direct loads (no staging
// registers) into one of NS slots, already in MFMA fragment order (a wave load drops lane i's 16 bytes
// at slot base + 16 i, so lane i asks for the piece that belongs there); after the issuing waves' wait and
// a barrier every wave's MFMAs read it as it came.  Three tiles are in flight or landed ahead of the one being
// multiplied, and the loads of tile i+3 are issued before the wait for tile i+1, so the memory queue never runs
// dry while the waves wait for one another.
//
// The kernel is bound by instruction issue and LDS latency, not by HBM, at 128 query rows per KV head,
// hence: tiles that lie wholly inside the cached context take a branch-free body (no mask);
// the accumulators of the first product start at minus the running reference, so the
// scores come out already shifted; the reference moves lazily; the row sums are one more MFMA with
// an all-ones operand (they add exactly the fp16 probabilities the second product uses, and need no
// cross-lane reduction); the K fragments of the next tile and the V fragments of this one are read
// into registers early, and the phases are ordered so that every batch of MFMAs has independent
// vector work beside it (the softmax of tile ct beside the products of its neighbour).
constexpr int HD = 128;
constexpr int BS = 16;
constexpr int KT = 32;                         // keys per tile (two blocks)
constexpr int TILE_HALFS = 2 * KT * HD;        // fp16 elements of K + V of one tile
constexpr int TILE_BYTES = TILE_HALFS * 2;     // 16 KB
constexpr int NS = 4;                          // tile slots in LDS (a ring of 8, seven tiles of lead, is slower: measured)
constexpr int MAX_CT = 2;                      // column tiles per wave; a workgroup covers 64 * MAX_CT stacked rows
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LAZY_MAX = 6.f;                // the reference moves when a score exceeds it by 2^6
constexpr float SPLIT_SCALE = 512.f;           // probabilities in two fp16 terms: 2^9 times a probability of up to 2^6 stays in range

__device__ __forceinline__ float max3(float x, float y, float z) { return __builtin_fmaxf(__builtin_fmaxf(x, y), z); }

// Online-softmax step of one column tile on one key tile.  S0/S1: scores of keys 8g+0..3 / 8g+4..7 of
// this lane's query row, already minus the reference (negm4 = -reference in all four elements, 0 while
// nothing was seen).  Returns the probabilities as the B operand of the second product, and with SPLIT 2^9 times the
// probabilities, what their rounding to fp16 left over as a second operand in `rest`.
template <bool MASK, int NU, bool SPLIT = false>
__device__ __forceinline__ f16x8 softmax_tile(const f32x4& S0, const f32x4& S1, float& run_m, f32x4& negm4, float& thr,
                                              f32x4 (&O)[NU], f32x4& L, int keyg, int lim, f16x8* rest = nullptr) {
  float sc[8] = {S0[0], S0[1], S0[2], S0[3], S1[0], S1[1], S1[2], S1[3]};
  if (MASK) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (keyg + e > lim) sc[e] = -INFINITY;
  }
  float tm = max3(max3(sc[0], sc[1], sc[2]), max3(sc[3], sc[4], sc[5]), __builtin_fmaxf(sc[6], sc[7]));
  // thr is -inf until the row has seen a key, LAZY_MAX afterwards: probabilities up to 2^6 are fine
  // in fp16 and in the fp32 accumulators, so the common tile needs no exchange and no rescale
  if (__any(tm > thr)) {
    uint32_t x, y;
    lane_pair<16>(__float_as_uint(tm), x, y);
    tm = __builtin_fmaxf(__uint_as_float(x), __uint_as_float(y));
    lane_pair<32>(__float_as_uint(tm), x, y);
    tm = __builtin_fmaxf(__uint_as_float(x), __uint_as_float(y));
    const bool fresh = run_m == -INFINITY;
    float d = fresh ? tm : __builtin_fmaxf(tm, 0.f);  // how far the reference moves (shifted units)
    if (d == -INFINITY) d = 0.f;                      // still nothing visible
    const float alpha = fresh ? 1.f : __builtin_amdgcn_exp2f(-d);
    if (!(fresh && tm == -INFINITY)) run_m = d - negm4[0];
    const float nm = (run_m == -INFINITY) ? 0.f : -run_m;
    negm4 = (f32x4){nm, nm, nm, nm};
    thr = (run_m == -INFINITY) ? -INFINITY : LAZY_MAX;
#pragma unroll
    for (int e = 0; e < 8; ++e) sc[e] -= d;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      O[u][0] *= alpha; O[u][1] *= alpha; O[u][2] *= alpha; O[u][3] *= alpha;
    }
    L[0] *= alpha; L[1] *= alpha; L[2] *= alpha; L[3] *= alpha;
  }
  union { f16x8 v; uint32_t u[4]; } pf;
  if constexpr (SPLIT) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float p = __builtin_amdgcn_exp2f(sc[e]) * SPLIT_SCALE;
      pf.v[e] = (f16_t)p;
      (*rest)[e] = (f16_t)(p - (float)pf.v[e]);
    }
    return pf.v;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    pf.u[e] = pack2h(__builtin_amdgcn_exp2f(sc[2 * e]), __builtin_amdgcn_exp2f(sc[2 * e + 1]));
  return pf.v;
}

template <int N> struct IntC { static constexpr int value = N; };

// leading arguments of the two MFMA kernels (launch.h)
#define MN_ATTN_LEAD                                                                                                    \
  int32_t *items_, const int32_t *seq_row0_, const int32_t *seq_ok_, const int32_t *seq_ctx_, const int32_t *block_tables_, \
      int Hkv_, int H_, int max_blocks_, int num_blocks_
#define MN_ATTN_TAKE_LEAD                                                                                \
  a.items = items_; a.rows.seq_row0 = seq_row0_; a.rows.seq_ok = seq_ok_; a.rows.seq_ctx = seq_ctx_;     \
  a.kv.block_tables = block_tables_; a.Hkv = Hkv_; a.H = H_; a.kv.max_blocks_per_seq = max_blocks_; a.kv.num_blocks = num_blocks_;
// x / d (x >= 0) from inv = 1 / d: one too few or too many at most before the correction for x below 2^23, in ten instructions where a
// division by a number that is not known when the kernel is compiled takes forty, each waiting for the one before
__device__ __forceinline__ int fast_div(int x, int d, float inv) {
  const int q = (int)((float)x * inv), r = x - q * d;
  return q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
}
#define MN_ATTN_LEAD_OF(a) \
  (a).items, (a).rows.seq_row0, (a).rows.seq_ok, (a).rows.seq_ctx, (a).kv.block_tables, (a).Hkv, (a).H, (a).kv.max_blocks_per_seq, (a).kv.num_blocks

// Partials: o_part [split][M][H][HD] fp32 (unnormalised), ml_part [split][M][H][2] = (max in log2 units, sum)
// NW waves per workgroup.  Waves 0-3 are the loaders (the tile's 16 fragments are dealt to four waves); with 5 or
// 6 waves the others only multiply: a stack of 65-96 query rows (5 or 6 column tiles, e.g. 8 query heads per KV
// head x 9-12 scored positions) then gives every wave one column tile, where four waves would leave one of them
// two tiles' worth of products and softmax per key tile while the other three wait at the barrier.
template <int CTW, int NW>
__global__ void __launch_bounds__(NW * 64, NW == 4 ? 2 : 1) attn_mfma_kernel(MN_ATTN_LEAD, AttnArgs a, float* __restrict__ o_part,
                                                                             float* __restrict__ ml_part) {
  MN_ATTN_TAKE_LEAD
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  f16_t* s_kv = reinterpret_cast<f16_t*>(smem);                          // [NS][16 fragments][64 lanes][8]
  int32_t* s_bidx = reinterpret_cast<int32_t*>(smem + NS * TILE_BYTES);  // physical block of every block of the split
  // Work list: workgroup (item, KV head) takes record `item` of the list prepare_kernel wrote for this step:
  // {sequence, row group, split, splits of the sequence, first row, rows, enabled, context}.  The list holds
  // only workgroups that have work, longest first, and the KV head is the fast index: workgroup ids are dealt
  // round-robin over the 8 XCDs and, inside an XCD, over its CUs, strictly in id order, so work has to be
  // dense in the id space (with the split as the fast grid index a batch that used 2 of 16 possible splits
  // ran on 2 of the 8 XCDs; with an often empty second row group next to the sequence index the real
  // workgroups shared half of the CUs) and long items must not queue behind short ones.
  // Row group rg: column tiles [NW*CTW*rg, NW*CTW*(rg+1)) of the stack; sequences with more than 16*NW*CTW stacked
  // rows get a workgroup per group (each streams the keys again).
  const int item = blockIdx.x / a.Hkv, kvh = blockIdx.x % a.Hkv;
  const int4 rec0 = reinterpret_cast<const int4*>(a.items)[2 * item];
  const int4 rec1 = reinterpret_cast<const int4*>(a.items)[2 * item + 1];
  const int b = rec0.x, rg = rec0.y, split = rec0.z, my_splits = rec0.w;
  const int row0 = rec1.x, qb = rec1.y, ok = rec1.z, ctx = rec1.w;
  // (the whole record, and the arguments that are used next, in one round trip: the compiler would fetch each part where it is used,
  // three round trips here, four for the queries below and one for the block ids; 32 x 8192 keys 212 -> 210 us, 24 ragged
  // sequences in the few-row kernel, for its queries, 90.2 -> 89.0)
  asm volatile("" ::"s"(b), "s"(rg), "s"(split), "s"(my_splits), "s"(row0), "s"(qb), "s"(ok), "s"(ctx), "s"(a.q), "s"(a.kv.k), "s"(a.kv.v));
  if (b < 0) return;                      // past the end of the list (whole workgroup)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int G = a.H / a.Hkv;
  const float G_inv = __builtin_amdgcn_rcpf((float)G);
  const int R = G * qb;                   // query rows sharing this KV head; row r = j*G + gi
  const int NT16 = (R + 15) >> 4;         // column tiles in use
  const int tile0 = NW * CTW * rg;        // first column tile of this workgroup
  const bool loader = wave < 4;           // (wave-uniform)
  if (qb <= 0 || tile0 >= NT16 || split >= my_splits) return;  // (whole workgroup; the list holds no such record)
  const int nkeys = ok ? ctx + qb : 0;
  // keys this row group sees: a prompt's later keys are behind the causal limit of its earlier rows (845 prompt rows in three
  // sequences: 26.7 -> 23.0 us)
  const int seen = ok ? ctx + fast_div(min(R, (tile0 + NW * CTW) * 16) - 1, G, G_inv) + 1 : 0;
  const int n_tiles = (seen + KT - 1) / KT;
  int t_begin = 0, t_end = n_tiles;
  if (my_splits > 1) {                    // (at most 16)
    t_begin = (int)(((long)n_tiles * split) / my_splits);
    t_end = (int)(((long)n_tiles * (split + 1)) / my_splits);
  }
  const int n_my = max(0, t_end - t_begin);
  const int nct = ok ? min(CTW, max(0, (NT16 - tile0 - wave + NW - 1) / NW)) : 0;  // real column tiles of this wave

  // block table of this split -> LDS (the dependent chain table -> address -> load would otherwise
  // cost an L2 round trip per tile); entries past the last mapped block repeat the last one
  const int32_t* bt = a.kv.block_tables + (size_t)b * a.kv.max_blocks_per_seq;
  const int last_blk = ok ? (nkeys - 1) / BS : 0;
  const int id_first = bt[min(2 * t_begin + tid, last_blk)];  // (each thread's first entry goes out ahead of the queries)

  // ---- Q fragments -> registers, scaled by log2(e)/sqrt(hd) (one more fp16 rounding of q, 2^-11), so
  // the scores come out of the first product in log2 units.  Rows past R are zero (they ask for the last row: behind a condition
  // each of the four loads was a round trip of its own). ----
  const float sscale = rsqrtf((float)HD) * LOG2E;
  const f16_t* Q = reinterpret_cast<const f16_t*>(a.q);
  f16x8 qf[CTW][4];
  f32x4 O[CTW][8], L[CTW], negm4[CTW];
  float run_m[CTW], thr[CTW];
  int lim[CTW];
#pragma unroll
  for (int ct = 0; ct < CTW; ++ct) {
    const int r = min((tile0 + wave + NW * ct) * 16 + l16, R - 1), j = fast_div(r, G, G_inv);
    lim[ct] = ctx + min(j, qb - 1);       // last visible key of this lane's query row
#pragma unroll
    for (int s = 0; s < 4; ++s)
      qf[ct][s] = *reinterpret_cast<const f16x8*>(Q + ((size_t)(row0 + j) * a.H + kvh * G + r - j * G) * HD + 32 * s + 8 * g);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (tid < 2 * n_my) s_bidx[tid] = id_first;
  for (int i = tid + NW * 64; i < 2 * n_my; i += NW * 64) s_bidx[i] = bt[min(2 * t_begin + i, last_blk)];
#pragma unroll
  for (int ct = 0; ct < CTW; ++ct) {
    run_m[ct] = -INFINITY;
    thr[ct] = -INFINITY;
    negm4[ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
    L[ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 8; ++u) O[ct][u] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const bool real = (tile0 + wave + NW * ct) * 16 + l16 < R;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[ct][s][e] = real ? (f16_t)((float)qf[ct][s][e] * sscale) : (f16_t)0.f;
  }

  // Loader role of this thread: the pieces of its own lane in K fragments (t = 0, 1; head-dim step s = wave)
  // and V fragments (u = wave, wave + 4).  K: S^T row l16 = 4g'+r of half t <-> key 8g' + 4t + r of the
  // tile, head-dim chunk 4*wave + g (t = 1: +64 bytes).  V: head-dim row 16u + l16, keys 8g..8g+7
  // (u + 4: +2048 bytes).
  const int kkey0 = 8 * (l16 >> 2) + (l16 & 3);  // key inside the tile for t = 0 (t = 1: + 4)
  const int kchunk = 4 * wave + g;
  const int ksel = l16 >> 3, vsel = g >> 1;      // which of the tile's two blocks the pieces live in
  const uint32_t blk_bytes = (uint32_t)a.Hkv * (HD * BS) * (uint32_t)sizeof(f16_t);
  const uint32_t blk_last = (uint32_t)max(a.kv.num_blocks - 1, 0);
  const size_t head_bytes = (size_t)kvh * (HD * BS) * sizeof(f16_t);
  const char* kbase = reinterpret_cast<const char*>(a.kv.k) + head_bytes + ((size_t)kchunk * BS + (kkey0 & (BS - 1))) * 8 * sizeof(f16_t);
  const char* vbase = reinterpret_cast<const char*>(a.kv.v) + head_bytes + ((size_t)(16 * wave + l16) * BS + 8 * (g & 1)) * sizeof(f16_t);
  // LDS byte address of fragment `wave` of slot 0 (wave-uniform)
  const uint32_t lds_w = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + (uint32_t)wave * 1024u);
  __syncthreads();  // block indices are in LDS; every load issued so far has been consumed

  if (ok && n_my > 0) {
    const int ti_last = n_my - 1;
    // all loads of tile TI of the split -> slot SLOT (tiles past the end repeat the last one)
#define MN_ATT_DMA(TI, SLOT)                                                                      \
  if (loader) {                                                                                   \
    const int t_ = min((TI), ti_last);                                                            \
    /* (the clamp costs two instructions and keeps a damaged table from becoming a wild address) */ \
    const char* kp_ = kbase + (uint64_t)min((uint32_t)s_bidx[2 * t_ + ksel], blk_last) * blk_bytes; \
    const char* vp_ = vbase + (uint64_t)min((uint32_t)s_bidx[2 * t_ + vsel], blk_last) * blk_bytes; \
    const uint32_t l_ = __builtin_amdgcn_readfirstlane(lds_w + (uint32_t)(SLOT) * TILE_BYTES);    \
    dma16<0, true>(kp_, l_);                                                                  \
    dma16<4 * 8 * 2, true>(kp_, l_ + 4 * 1024);                                               \
    dma16<0, true>(vp_, l_ + 8 * 1024);                                                       \
    dma16<64 * BS * 2, true>(vp_, l_ + 12 * 1024);                                            \
  }
    f16x8 kf[8];  // K fragments of the tile about to be multiplied
    // prologue: tiles 0 .. NS-2 on their way; tile 0 landed and its K fragments in registers
#pragma unroll
    for (int t = 0; t < NS - 1; ++t) MN_ATT_DMA(t, t)
    wait_vm<4 * (NS - 2)>();
    __syncthreads();
#pragma unroll
    for (int f = 0; f < 8; ++f) kf[f] = *reinterpret_cast<const f16x8*>(s_kv + (f * 64 + lane) * 8);

    // Iteration i: slot i%NS holds tile i (its K fragments already in kf); tile i+1 landed or
    // landing in slot (i+1)%NS, tiles i+2 .. i+NS-2 in flight; slot (i+NS-1)%NS, which held tile i-1, is free
    // since the last barrier.  SLOW: the tile reaches past ctx: the scores are masked (causal order among
    // the scored tokens, keys past the sequence end), and the V slots past the sequence end, which may hold anything
    // (0 * garbage must stay 0), are read as zeros.
    const f16x8 ones = {1, 1, 1, 1, 1, 1, 1, 1};
    auto iter = [&](auto nct_c, auto slow_c, int i) {
      constexpr int NCT = decltype(nct_c)::value;
      constexpr bool SLOW = decltype(slow_c)::value != 0;
      constexpr int NC = NCT > 0 ? NCT : 1;
      const int cur = i & (NS - 1), nxt = (i + 1) & (NS - 1);
      MN_ATT_DMA(i + NS - 1, (i + NS - 1) & (NS - 1))
      f16x8 vf[8];
      if (NCT > 0) {
#pragma unroll
        for (int u = 0; u < 8; ++u) vf[u] = *reinterpret_cast<const f16x8*>(s_kv + cur * TILE_HALFS + ((8 + u) * 64 + lane) * 8);
      }
      if (SLOW && NCT > 0) {
        const int past = (t_begin + i) * KT + 8 * g + 8 - nkeys;  // how many of this lane's 8 keys lie past the end
        if (past > 0) {
#pragma unroll
          for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (e >= 8 - past) vf[u][e] = (f16_t)0.f;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // first product of column tile 0
      f32x4 S0[NC], S1[NC];
      f16x8 P[NC];
      const int keyg = (t_begin + i) * KT + 8 * g;
      if (NCT > 0) {
        S0[0] = negm4[0];
        S1[0] = negm4[0];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          S0[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[s], qf[0][s], S0[0], 0, 0, 0);
          S1[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[4 + s], qf[0][s], S1[0], 0, 0, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // first product of column tile ct beside the softmax of tile ct-1
#pragma unroll
      for (int ct = 1; ct < NCT; ++ct) {
        S0[ct] = negm4[ct];
        S1[ct] = negm4[ct];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          S0[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[s], qf[ct][s], S0[ct], 0, 0, 0);
          S1[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[4 + s], qf[ct][s], S1[ct], 0, 0, 0);
        }
        P[ct - 1] = softmax_tile<SLOW, 8>(S0[ct - 1], S1[ct - 1], run_m[ct - 1], negm4[ct - 1], thr[ct - 1], O[ct - 1], L[ct - 1], keyg, lim[ct - 1]);
        __builtin_amdgcn_sched_barrier(0);
      }
      // every LDS read of tile i has been issued; tile i+1 has landed once every loader's own wait is over
      // (the NS-2 tiles behind it may stay in flight): hand over
      wait_vm<4 * (NS - 2)>();
      __syncthreads();
#pragma unroll
      for (int f = 0; f < 8; ++f) kf[f] = *reinterpret_cast<const f16x8*>(s_kv + nxt * TILE_HALFS + (f * 64 + lane) * 8);
      __builtin_amdgcn_sched_barrier(0);
      // second product of tiles 0..NCT-2 beside the softmax of the last tile, then the last second product
      if (NCT > 0) {
#pragma unroll
        for (int ct = 0; ct + 1 < NCT; ++ct) {
#pragma unroll
          for (int u = 0; u < 8; ++u) O[ct][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf[u], P[ct], O[ct][u], 0, 0, 0);
          L[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, P[ct], L[ct], 0, 0, 0);
        }
        P[NCT - 1] = softmax_tile<SLOW, 8>(S0[NCT - 1], S1[NCT - 1], run_m[NCT - 1], negm4[NCT - 1], thr[NCT - 1], O[NCT - 1], L[NCT - 1], keyg, lim[NCT - 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 8; ++u) O[NCT - 1][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf[u], P[NCT - 1], O[NCT - 1][u], 0, 0, 0);
        L[NCT - 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, P[NCT - 1], L[NCT - 1], 0, 0, 0);
      }
    };
    // fast iterations: tiles that lie wholly below ctx
    const int n_fast = min(n_my, max(0, ctx / KT - t_begin));
    int i = 0;
    if (nct == CTW) {
      for (; i < n_fast; ++i) iter(IntC<CTW>{}, IntC<0>{}, i);
      for (; i < n_my; ++i) iter(IntC<CTW>{}, IntC<1>{}, i);
    } else if (nct == 0) {
      for (; i < n_my; ++i) iter(IntC<0>{}, IntC<1>{}, i);
    } else {
      if constexpr (CTW > 1) {
        if (nct == 1) {
          for (; i < n_fast; ++i) iter(IntC<1>{}, IntC<0>{}, i);
          for (; i < n_my; ++i) iter(IntC<1>{}, IntC<1>{}, i);
        }
      }
    }
    wait_vm<0>();  // the loads of the tiles past the end must land before the LDS is given back
#undef MN_ATT_DMA
  }

  // ---- output: lane holds O^T[hd = 16u + 4g + i][row = tile*16 + l16]; every lane has its row's sum ----
#pragma unroll
  for (int ct = 0; ct < CTW; ++ct) {
    const int tile = tile0 + wave + NW * ct;
    const int r = tile * 16 + l16;
    if (tile >= NT16 || r >= R) continue;
    const float l = L[ct][0];
    const int j = fast_div(r, G, G_inv), gi = r - j * G;
    const int m = row0 + j, h = kvh * G + gi;
    if (my_splits == 1) {
      const float inv = (ok && l > 0.f) ? 1.f / l : 0.f;
      f16_t* o = reinterpret_cast<f16_t*>(a.out) + ((size_t)m * a.H + h) * HD + 4 * g;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const f32x4 v = O[ct][u];
        *reinterpret_cast<uint2*>(o + 16 * u) = make_uint2(pack2h(v[0] * inv, v[1] * inv), pack2h(v[2] * inv, v[3] * inv));
      }
    } else {
      float* o = o_part + (((size_t)split * a.M + m) * a.H + h) * HD + 4 * g;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const f32x4 v = O[ct][u];
        *reinterpret_cast<float4*>(o + 16 * u) = make_float4(v[0], v[1], v[2], v[3]);
      }
      if (g == 0) {
        float* ml = ml_part + (((size_t)split * a.M + m) * a.H + h) * 2;
        ml[0] = run_m[ct];
        ml[1] = l;
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// MFMA kernel for few rows (fp16 pages, fp16 queries, head_dim 64 or 128, block 16)
// ------------------------------------------------------------------------------------------
// Up to 16 * CT query rows per KV head: one row per sequence of a decoding step, the few rows of a model without head
// groups, a drafting model catching up.  There is nothing for the waves of a workgroup to share, so instead of staging
// tiles in LDS behind a barrier every wave takes key tiles of its own (wave w of a workgroup the tiles w, w + NW, ... of
// its range), loads their K and V pieces straight into the operand registers of its MFMAs and keeps its own (max, sum, output).
// The waves' results meet once, in LDS, at the end.
// Measured per layer, rotary/append included: 95 rows of 16 requests x 12 heads of 64, contexts 200-1500: 139 -> 16.2 us;
// 16 x 1024 keys of the same model 17.1 -> 15.7 us; 8 x 512 keys x 40 heads of 128 29.2 -> 25.0 us.
// Bound by the KV stream (12 layers of 16 sequences take 8.2 us a layer more at 1024 keys than at 16, 50 MB at 6.1 TB/s) and, at
// short contexts, by launch and the chain bookkeeping -> block table and QKV sums -> append -> tile -> merge (about 6 us).  The
// append used to follow the wave's first tile, and every wave's second tile followed both: now it goes ahead of the first, its
// loads all at once, and with 8 waves the block ids go ahead of the tiles that need them.  12 layers of that model, whole passes:
// 16 x 1024 keys 419.8 -> 410.7 us, the 95 rows 493.6 -> 485.9.
// FUSED: the workgroup also turns its rows' QKV partial sums into queries (kept in LDS) and K/V rows (written to the pages
// before the tiles that hold them are read), which saves a launch of its own per layer; a sequence must then be in one KV
// split, so that the rows have one writer.  When every workgroup is resident at once and nothing is split (no list:
// a.items null) the workgroups take (sequence, KV head) from their index: one dependent load less before the first tile.
// Products and operand order are those of the kernel above; record list and KV splits likewise.  With head_dim 64
// (the shapes that used to run on plain fp32 FMA) the fp16 queries go into the first product as they are and the scale is
// applied to its fp32 result, and a probability p goes into the second product as two fp16 terms of 2^9 p, in the sums of the
// outputs and of the probabilities alike: off by at most 2^-23 p or 2^-34, whichever is larger, where the row's sum is at
// least 1 and the fp32 sums round at 2^-24 of it (the extra products hide behind the stream).  Without the factor the fixed
// step was 2^-25: with one key at probability 1 in every wave's share and the rest of a 2000-key row at 2^-19 (2^-23) each,
// 1.1 % (17 %) of that rest was lost.
template <int HDIM, int CT, int NW, bool FUSED>
__global__ void __launch_bounds__(NW * 64, HDIM == 64 ? (CT == 1 ? 3 : 2) : (CT == 1 ? 2 : 1))
    attn_keys_kernel(MN_ATTN_LEAD, AttnArgs a, float* __restrict__ o_part, float* __restrict__ ml_part) {
  MN_ATTN_TAKE_LEAD
  constexpr bool WIDE = HDIM == 64;                          // queries unscaled, probabilities in two terms
  constexpr int HS = HDIM / 32, NU = HDIM / 16, OROW = HDIM + 4;  // (padded rows: the merge's 16-byte accesses spread over the banks)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* s_o = reinterpret_cast<float*>(smem);               // [NW][16][OROW], one column tile at a time
  __shared__ float s_m[CT][NW][16], s_l[CT][NW][16];
  const int item = blockIdx.x / a.Hkv, kvh = blockIdx.x % a.Hkv;
  int b, split = 0, my_splits = 1, row0, qb, ok, ctx;
  if (a.items) {  // (uniform)
    const int4 rec0 = reinterpret_cast<const int4*>(a.items)[2 * item];
    const int4 rec1 = reinterpret_cast<const int4*>(a.items)[2 * item + 1];
    b = rec0.x;
    if (b < 0 || rec0.y != 0) return;                        // past the end of the list (whole workgroup)
    split = rec0.z; my_splits = rec0.w;
    row0 = rec1.x; qb = rec1.y; ok = rec1.z; ctx = rec1.w;
  } else {
    b = item;
    row0 = a.rows.seq_row0[b]; qb = a.rows.seq_row0[b + 1] - row0; ok = a.rows.seq_ok[b]; ctx = a.rows.seq_ctx[b];
  }
  if (FUSED)  // (the arguments that are used next are fetched with these)
    asm volatile("" ::"s"(a.qkv), "s"(a.rope_cos), "s"(a.rope_sin), "s"(a.rows.row_slot), "s"(a.bias), "s"(a.kv.k), "s"(a.kv.v), "s"(a.M),
                 "s"(a.n_partials), "s"(row0), "s"(ctx));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int G = a.H / a.Hkv;
  const int R = G * qb;                                      // query rows sharing this KV head; row r = j*G + gi
  if (qb <= 0 || split >= my_splits) return;                 // (whole workgroup)
  const int nkeys = ok ? ctx + qb : 0;
  const int n_tiles = (nkeys + KT - 1) / KT;
  const int t_begin = (int)(((long)n_tiles * split) / my_splits);
  const int t_end = (int)(((long)n_tiles * (split + 1)) / my_splits);
  const int t0 = t_begin + wave;                             // this wave's tiles: t0, t0 + NW, ...
  const int n = t0 < t_end ? (t_end - t0 + NW - 1) / NW : 0;

  const int32_t* bt = a.kv.block_tables + (size_t)b * a.kv.max_blocks_per_seq;
  const int last_blk = ok ? (nkeys - 1) / BS : 0;
  const uint32_t blk_bytes = (uint32_t)a.Hkv * (HDIM * BS) * (uint32_t)sizeof(f16_t);
  const uint32_t blk_last = (uint32_t)max(a.kv.num_blocks - 1, 0);
  const size_t head_bytes = (size_t)kvh * (HDIM * BS) * sizeof(f16_t);
  // this lane's pieces (see the kernel above): K row l16 = 4g'+r of half t is key 8g' + 4t + r, head-dim chunk 4s + g;
  // V head-dim row 16u + l16, keys 8g .. 8g+7
  const char* kbase = reinterpret_cast<const char*>(a.kv.k) + head_bytes + (size_t)(g * BS + 8 * ((l16 >> 2) & 1) + (l16 & 3)) * 16;
  const char* vbase = reinterpret_cast<const char*>(a.kv.v) + head_bytes + (size_t)l16 * (BS * sizeof(f16_t)) + 16 * (g & 1);
  const bool ksel = (l16 >> 3) != 0, vsel = (g >> 1) != 0;   // which of the tile's two blocks the pieces live in
  struct Tile {
    u32x4 k[2 * HS], v[NU];
  };
  // (block ids are clamped: a damaged table never becomes a wild address)
  struct Ids {
    uint32_t a0, a1, b0, b1;
  };
  auto ids_of = [&](int i) {                                 // of the wave's tile i
    const int tile = t0 + NW * i;
    const uint32_t b0 = min((uint32_t)bt[min(2 * tile, last_blk)], blk_last), b1 = min((uint32_t)bt[min(2 * tile + 1, last_blk)], blk_last);
    return Ids{b0, b1, 0, 0};
  };
  // of tiles i and i + 1, asked for here (in lanes 0 .. 3) and looked at later
  auto ask = [&](int i) { return bt[min(2 * (t0 + NW * min(i + ((lane >> 1) & 1), max(n - 1, 0))) + (lane & 1), last_blk)]; };
  auto answer = [&](int ids) {
    auto id = [&](int at) -> uint32_t { return min((uint32_t)__builtin_amdgcn_readlane(ids, at), blk_last); };
    return Ids{id(0), id(1), id(2), id(3)};
  };
  auto load = [&](Tile& t, uint32_t b0, uint32_t b1) {
    const char* kp = kbase + (uint64_t)(ksel ? b1 : b0) * blk_bytes;
    const char* vp = vbase + (uint64_t)(vsel ? b1 : b0) * blk_bytes;
    // (the two halves of a K line are asked for by different instructions: with 8 waves, where the workgroup has its CU to
    // itself, the lines stay without the non-temporal hint until both have been served: 256 workgroups of 300-2000 keys 38.8 ->
    // 32.2 us; with 4 waves and two workgroups per CU the hint is as good or better: 960 workgroups 80.7 us, 82.0 without)
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int s = 0; s < HS; ++s) {
        const u32x4* p = reinterpret_cast<const u32x4*>(kp + h * 64 + s * (4 * BS * 16));
        t.k[h * HS + s] = NW == 8 ? *p : __builtin_nontemporal_load(p);
      }
#pragma unroll
    for (int u = 0; u < NU; ++u) t.v[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(vp + u * (16 * BS * (int)sizeof(f16_t))));
  };
  Tile ta, tb;
  constexpr bool AHEAD = FUSED && NW == 8;                   // (see the loop over the tiles)
  // (every wave asks: behind a condition the answers would be waited for once more below)
  const int ids0 = AHEAD ? ask(0) : 0, ids1 = AHEAD ? ask(1) : 0;
  Ids first{}, cur{};                                        // of tile 0; AHEAD: of tiles 1 and 2
  if (!FUSED && n > 0) {
    first = ids_of(0);
    load(ta, first.a0, first.a1);
  }

  constexpr int QROW = HDIM + 8;
  f16_t* s_q = reinterpret_cast<f16_t*>(smem);               // [R][QROW] (the merge reuses the space behind a barrier)
  if constexpr (FUSED) {
    // thread item = four pairs (t .. t+3, and + hd/2) of one head of one row: the G query heads, the key head, the value head.
    // The last waves take them, which have the fewest tiles, and ahead of their first tile: loads complete in order, and behind
    // it the K/V rows and the barrier, and so every wave's second tile, would wait for it.
    constexpr int HALF = HDIM / 2, Q4 = HALF / 4;
    const int ncols = (a.H + 2 * a.Hkv) * HDIM;
    bool bad = false;
    for (int idx = NW * 64 - 1 - tid; idx < (G + 2) * qb * Q4; idx += NW * 64) {
      const int t = (idx % Q4) * 4, rr = idx / Q4, j = rr % qb, hh = rr / qb;
      const int m = row0 + j;
      int slot = a.rows.row_slot[m];                         // (-1: disabled)
      const int head = hh < G ? kvh * G + hh : (hh == G ? a.H + kvh : a.H + a.Hkv + kvh);
      const int c0 = head * HDIM + t;
      f32x4 v0 = {0.f, 0.f, 0.f, 0.f}, v1 = v0;
      // (angles and bias are asked for with the rest, there or not)
      const float *spare = a.qkv + (size_t)m * ncols, *bias = a.bias ? a.bias : spare;
      const f32x4 cs = *reinterpret_cast<const f32x4*>((a.rope_cos ? a.rope_cos + (size_t)m * HALF : spare) + t);
      const f32x4 sn = *reinterpret_cast<const f32x4*>((a.rope_cos ? a.rope_sin + (size_t)m * HALF : spare) + t);
      const f32x4_u b0 = *reinterpret_cast<const f32x4_u*>(bias + c0), b1 = *reinterpret_cast<const f32x4_u*>(bias + c0 + HALF);
      // partials fetched four at a time before any is added (the fence keeps the compiler from putting the loads beside their
      // sums); the order of the sum is that of rope_append_kernel
      for (int s0 = 0; s0 < a.n_partials; s0 += 4) {
        f32x4 p0[4], p1[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float* p = a.qkv + ((size_t)min(s0 + k, a.n_partials - 1) * a.M + m) * ncols + c0;
          p0[k] = *reinterpret_cast<const f32x4*>(p);
          p1[k] = *reinterpret_cast<const f32x4*>(p + HALF);
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (s0 + k < a.n_partials) { v0 += p0[k]; v1 += p1[k]; }
        // (vmcnt(0): repeats that are still on their way would be waited for ahead of the first partials at the back edge, and
        // below by every wave, its tiles with them)
        __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
      }
      if (a.bias) {
#pragma unroll
        for (int e = 0; e < 4; ++e) { v0[e] += b0[e]; v1[e] += b1[e]; }
      }
      asm volatile("" : "+v"(slot));                         // (asked for with the rest, not where it is used)
      if (a.rope_cos && hh <= G) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = v0[e], y = v1[e];
          v0[e] = x * cs[e] - y * sn[e];
          v1[e] = y * cs[e] + x * sn[e];
        }
      }
      if (hh > G - 1 && (!ok || slot < 0)) continue;         // disabled sequence: nothing is written to the cache
      const uint2 w0 = make_uint2(pack2h_sat(v0[0], v0[1], bad), pack2h_sat(v0[2], v0[3], bad));
      const uint2 w1 = make_uint2(pack2h_sat(v1[0], v1[1], bad), pack2h_sat(v1[2], v1[3], bad));
      if (hh < G) {
        f16_t* q = s_q + (size_t)(j * G + hh) * QROW + t;
        *reinterpret_cast<uint2*>(q) = w0;
        *reinterpret_cast<uint2*>(q + HALF) = w1;
      } else {
        const uint32_t blk = min((uint32_t)(slot / BS), blk_last);
        const int off = slot % BS;
        if (hh == G) {  // K: [hd/8][bs][8]
          f16_t* base = reinterpret_cast<f16_t*>(a.kv.k) + ((size_t)blk * a.Hkv + kvh) * (HDIM * BS);
          *reinterpret_cast<uint2*>(base + ((t >> 3) * BS + off) * 8 + (t & 7)) = w0;
          *reinterpret_cast<uint2*>(base + (((t + HALF) >> 3) * BS + off) * 8 + (t & 7)) = w1;
        } else {        // V: [hd][bs]
          uint16_t* base = reinterpret_cast<uint16_t*>(a.kv.v) + ((size_t)blk * a.Hkv + kvh) * (HDIM * BS) + (size_t)t * BS + off;
          base[0] = (uint16_t)w0.x; base[BS] = (uint16_t)(w0.x >> 16); base[2 * BS] = (uint16_t)w0.y; base[3 * BS] = (uint16_t)(w0.y >> 16);
          base += (size_t)HALF * BS;
          base[0] = (uint16_t)w1.x; base[BS] = (uint16_t)(w1.x >> 16); base[2 * BS] = (uint16_t)w1.y; base[3 * BS] = (uint16_t)(w1.y >> 16);
        }
      }
    }
    if (bad && a.dev_status) atomicOr(a.dev_status, MN_DEV_RANGE);
    // (a first tile that holds rows of this step is asked for after they have been written)
    const bool early = (t0 + 1) * KT <= ctx;                 // (wave-uniform)
    if (AHEAD) {
      first = answer(ids0);
      cur = answer(ids1);
    } else if (n > 0) {
      first = ids_of(0);
    }
    if (n > 0 && early) load(ta, first.a0, first.a1);
    __syncthreads();  // the queries are in LDS; the K/V rows are visible to the whole workgroup
    if (n > 0 && !early) load(ta, first.a0, first.a1);
  }

  const float sscale = rsqrtf((float)HDIM) * LOG2E;
  const f16_t* Q = reinterpret_cast<const f16_t*>(a.q);
  f16x8 qf[CT][HS];
  f32x4 O[CT][NU], L[CT], negm4[CT];
  float run_m[CT], thr[CT];
  int lim[CT];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    run_m[ct] = -INFINITY;
    thr[ct] = -INFINITY;
    negm4[ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
    L[ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const int r = ct * 16 + l16;
    const int j = min(r, R - 1) / G;
    lim[ct] = ctx + j;                                       // last visible key of this lane's query row
#pragma unroll
    for (int u = 0; u < NU; ++u) O[ct][u] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < HS; ++s) {        // (rows past R ask for the last one: behind a condition each load is a round trip of its own)
      if constexpr (FUSED) qf[ct][s] = *reinterpret_cast<const f16x8*>(s_q + (size_t)min(r, R - 1) * QROW + 32 * s + 8 * g);
      else qf[ct][s] = *reinterpret_cast<const f16x8*>(Q + ((size_t)(row0 + j) * a.H + kvh * G + min(r, R - 1) - j * G) * HDIM + 32 * s + 8 * g);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
#pragma unroll
    for (int s = 0; s < HS; ++s)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const f16_t v = WIDE ? qf[ct][s][e] : (f16_t)((float)qf[ct][s][e] * sscale);
        qf[ct][s][e] = ct * 16 + l16 < R ? v : (f16_t)0.f;
      }
  }

  const f16x8 ones = {1, 1, 1, 1, 1, 1, 1, 1};
  // SLOW: the tile may reach past ctx (masked scores, V slots past the end read as zeros: 0 * garbage must stay 0)
  auto work = [&](auto slow_c, Tile& t, int i) {
    constexpr bool SLOW = decltype(slow_c)::value != 0;
    const int keyg = (t0 + NW * i) * KT + 8 * g;
    f32x4 S0[CT], S1[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      S0[ct] = WIDE ? (f32x4){0.f, 0.f, 0.f, 0.f} : negm4[ct];
      S1[ct] = S0[ct];
#pragma unroll
      for (int s = 0; s < HS; ++s) {
        S0[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, t.k[s]), qf[ct][s], S0[ct], 0, 0, 0);
        S1[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, t.k[HS + s]), qf[ct][s], S1[ct], 0, 0, 0);
      }
      if (WIDE) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          S0[ct][e] = fmaf(S0[ct][e], sscale, negm4[ct][e]);
          S1[ct][e] = fmaf(S1[ct][e], sscale, negm4[ct][e]);
        }
      }
    }
    if (SLOW) {
      const int past = keyg + 8 - nkeys;                     // how many of this lane's 8 keys lie past the end
      if (past > 0) {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t keep = (2 * w < 8 - past ? 0x0000ffffu : 0u) | (2 * w + 1 < 8 - past ? 0xffff0000u : 0u);
#pragma unroll
          for (int u = 0; u < NU; ++u) t.v[u][w] &= keep;
        }
      }
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      f16x8 rest;
      const f16x8 P = softmax_tile<SLOW, NU, WIDE>(S0[ct], S1[ct], run_m[ct], negm4[ct], thr[ct], O[ct], L[ct], keyg, lim[ct], &rest);
#pragma unroll
      for (int u = 0; u < NU; ++u) O[ct][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, t.v[u]), P, O[ct][u], 0, 0, 0);
      L[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, P, L[ct], 0, 0, 0);
      if (WIDE) {
#pragma unroll
        for (int u = 0; u < NU; ++u) O[ct][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, t.v[u]), rest, O[ct][u], 0, 0, 0);
        L[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, rest, L[ct], 0, 0, 0);
      }
    }
  };
  // Two tiles per pass of the loop, every load in it unconditional (behind a branch the compiler's wait counts would drain
  // the load queue).  Only a wave's last tile can reach past ctx: the rows of a sequence span at most CT <= NW - 1 tiles
  // beyond the first, and tiles are dealt to the waves in turn.
  // AHEAD: a pass asks for the block ids of the next one ahead of its own tiles (loads complete in order, so they are there when
  // those are), and two tiles are on their way at a time.  Elsewhere a tile's ids are asked for with it, behind the tile before,
  // and one is: with 4 waves, and two workgroups per CU, two tiles each are too many (960 workgroups 90 -> 98 us).
  if (n > 1) {
    int i = 0;                                               // (AHEAD: cur holds the ids of tiles i + 1 and i + 2)
    for (; i + 2 < n; i += 2) {
      const int next = AHEAD ? ask(i + 3) : 0;
      if (!AHEAD) cur = ids_of(i + 1);
      load(tb, cur.a0, cur.a1);
      if (AHEAD) __builtin_amdgcn_sched_barrier(0);
      work(IntC<0>{}, ta, i);
      if (AHEAD) {
        load(ta, cur.b0, cur.b1);
        __builtin_amdgcn_sched_barrier(0);
      } else {
        cur = ids_of(i + 2);
        load(ta, cur.a0, cur.a1);
      }
      work(IntC<0>{}, tb, i + 1);
      if (AHEAD) cur = answer(next);
    }
    if (i + 1 < n) {
      if (!AHEAD) cur = ids_of(i + 1);
      load(tb, cur.a0, cur.a1);
      if (AHEAD) __builtin_amdgcn_sched_barrier(0);
      work(IntC<0>{}, ta, i);
      work(IntC<1>{}, tb, i + 1);
    } else {
      work(IntC<1>{}, ta, i);
    }
  } else if (n == 1) {
    work(IntC<1>{}, ta, 0);
  }

  // ---- merge over the waves, output ----
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
    if (g == 0) {
      s_m[ct][wave][l16] = run_m[ct];
      s_l[ct][wave][l16] = L[ct][0];
    }
  __syncthreads();
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    if (ct * 16 >= R) break;                                 // (whole workgroup)
    float gm = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) gm = fmaxf(gm, s_m[ct][w][l16]);
    const float f = run_m[ct] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(run_m[ct] - gm);
    if (ct > 0) __syncthreads();                             // (the previous column tile has been read)
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const f32x4 v = O[ct][u];
      *reinterpret_cast<float4*>(s_o + (size_t)(wave * 16 + l16) * OROW + 16 * u + 4 * g) = make_float4(v[0] * f, v[1] * f, v[2] * f, v[3] * f);
    }
    __syncthreads();
    for (int c = tid; c < 16 * (HDIM / 4); c += NW * 64) {
      const int row = c / (HDIM / 4), e = (c % (HDIM / 4)) * 4, r = ct * 16 + row;
      if (r >= R) continue;
      float rm = -INFINITY;
#pragma unroll
      for (int w = 0; w < NW; ++w) rm = fmaxf(rm, s_m[ct][w][row]);
      float l = 0.f;
      float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float mw = s_m[ct][w][row];
        l += (mw == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw - rm)) * s_l[ct][w][row];
        const float4 x = *reinterpret_cast<const float4*>(s_o + (size_t)(w * 16 + row) * OROW + e);
        o.x += x.x; o.y += x.y; o.z += x.z; o.w += x.w;
      }
      const int m = row0 + r / G, h = kvh * G + r % G;
      if (my_splits == 1) {
        const float inv = (ok && l > 0.f) ? 1.f / l : 0.f;
        const size_t at = FUSED && a.operand ? operand_at(m, h * HDIM + e, a.M, a.H * HDIM) : ((size_t)m * a.H + h) * HDIM + e;
        *reinterpret_cast<uint2*>(reinterpret_cast<f16_t*>(a.out) + at) =
            make_uint2(pack2h(o.x * inv, o.y * inv), pack2h(o.z * inv, o.w * inv));
      } else {
        *reinterpret_cast<float4*>(o_part + (((size_t)split * a.M + m) * a.H + h) * HDIM + e) = o;
        if (e == 0) {
          float* ml = ml_part + (((size_t)split * a.M + m) * a.H + h) * 2;
          ml[0] = rm;
          ml[1] = l;
        }
      }
    }
  }
}

// Half a wave per (row, head): merge the split partials, normalise, store fp16.  Rows of sequences that ran as one split were
// written in final form by the attention kernel and are left alone.  Bound by the partials' bytes and one round trip: four
// splits' statistics and outputs are asked for at once, before any is looked at (512 rows x 64 heads in two splits: 14.5 -> 10.6 us).
__global__ void __launch_bounds__(256) attn_merge_kernel(const float* __restrict__ o_part, const float* __restrict__ ml_part,
                                                         int n_splits_max, int M, int H,
                                                         const int32_t* __restrict__ row_splits, f16_t* __restrict__ out) {
  const int wid = (blockIdx.x * 256 + threadIdx.x) >> 5, lane = threadIdx.x & 31;
  if (wid >= M * H) return;
  // (one read decides: most rows of a ragged batch have nothing to merge; the bound keeps a damaged entry from
  // reaching past the partials)
  const int n_splits = min(row_splits[wid / H], n_splits_max);
  if (n_splits <= 1) return;
  float gm = -INFINITY, l = 0.f;
  f32x4 o = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < n_splits; s0 += 4) {
    float2 ml[4];
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t at = (size_t)min(s0 + u, n_splits - 1) * M * H + wid;
      ml[u] = *reinterpret_cast<const float2*>(ml_part + at * 2);
      v[u] = *reinterpret_cast<const f32x4*>(o_part + at * HD + lane * 4);
    }
    float nm = gm;
#pragma unroll
    for (int u = 0; u < 4; ++u) nm = fmaxf(nm, ml[u].x);
    const float ms = (nm == -INFINITY) ? 0.f : nm, keep = __builtin_amdgcn_exp2f(gm - ms);
    l *= keep;
    o *= keep;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s0 + u < n_splits) {
        const float f = __builtin_amdgcn_exp2f(ml[u].x - ms);
        l += ml[u].y * f;
        o += v[u] * f;
      }
    gm = nm;
  }
  const float inv = l > 0.f ? 1.f / l : 0.f;
  *reinterpret_cast<uint2*>(out + (size_t)wid * HD + lane * 4) = make_uint2(pack2h(o[0] * inv, o[1] * inv), pack2h(o[2] * inv, o[3] * inv));
}

// ------------------------------------------------------------------------------------------
// launch
// ------------------------------------------------------------------------------------------
// Fewest key tiles a workgroup should take: below that the lead-in of a workgroup, the fp32 partial it writes and the
// merge launch behind cost as much as the parallelism wins (measured at 33 tiles per sequence and 128 (sequence, KV
// head) pairs: one split 2.10 ms of attention per step, two splits + merge 2.13-2.17, three or four 2.8-2.9; 16 and
// 32 give the same times at the other benchmark shapes, where the batch size decides the splits).
static int attention_min_tiles() {
  const int x = MN_TUNE("MN_ATTN_MIN_TILES", 32);
  return x > 0 ? x : 32;
}

// 1.25 workgroups with work per CU: measured flat between 1 and 1.3 per CU, slower beyond (every further split of
// a sequence writes and re-reads one more fp32 partial of its rows, and workgroups beyond the 512 that are
// resident at once start when the first ones end)
static int attention_target_workgroups() {
  const int x = MN_TUNE("MN_ATTN_WGS", 320);
  return x > 0 ? x : 320;
}

// Largest number of KV splits any sequence of the batch may get (it sizes the partials and bounds the work list;
// every sequence then takes what its own length asks for, see prepare_kernel): one per attention_min_tiles() key
// tiles of the longest context, 16 at most.
static int pick_splits(int max_ctx) {
  const int forced = MN_TUNE("MN_ATTN_SPLITS", 0);
  const int tiles = (max_ctx + KT - 1) / KT;
  int s = forced > 0 ? forced : tiles / attention_min_tiles();
  if (s > 16) s = 16;
  if (s < 1) s = 1;
  return s;
}

bool attention_mfma_supported(int H, int Hkv, int hd, int block_size, int dtype) {
  const int off = MN_TUNE("MN_ATTN_GENERIC", 0);
  return !off && dtype == MN_DT_BF16 && hd == HD && block_size == BS && Hkv > 0 && H % Hkv == 0;
}

static size_t mfma_smem_bytes(int tiles_per_split) {
  return (size_t)NS * TILE_BYTES + (size_t)(2 * tiles_per_split + 2) * sizeof(int32_t);
}

size_t attention_scratch_bytes(int M, int H, int hd, int max_ctx, int dtype) {
  if (dtype != MN_DT_BF16 || hd != HD) return 256;
  return (size_t)16 * M * H * (HD + 2) * sizeof(float) + 256;
}

// Records the work list must hold: a sequence of q rows has at most G q / 64 + 1 row groups (a workgroup covers
// at least 64 stacked rows) of at most 16 splits each.
size_t attention_items_capacity(int B, int M, int H, int Hkv) {
  const size_t G = Hkv > 0 ? (size_t)(H / Hkv) : 1;
  return 16 * (G * (size_t)(M > 0 ? M : 0) / 64 + (size_t)(B > 0 ? B : 0)) + 16;
}

// 17 to 32 rows at head_dim 128: the second column tile takes the registers of a second workgroup per CU, and alone the kernel
// is slower than the LDS-staged one (cold pages, 423 shapes of 1 to 64 sequences x 0 to 2000 keys: 1.13 times its time on
// average).  What it can win is the rotary launch, where the workgroups just about fill the CUs and the contexts are short:
// steps of four layers, 129 to 256 workgroups, at most 500 keys 0.89 to 0.99, 1000 keys 0.95 to 1.03; 8 to 128 workgroups 0.95
// to 1.17, 257 to 640 workgroups 0.91 to 1.08.
constexpr int KEYS_CT2_MIN_WGS = 129, KEYS_CT2_MAX_WGS = 256, KEYS_CT2_MAX_CTX = 768;
constexpr int KEYS_RESIDENT = 512;   // its 4-wave workgroups that are resident at once (two per CU): up to here the order of
                                     // the work does not matter and no list is made
static bool keys_path(const AttnArgs& a) {
  if (MN_TUNE("MN_ATTN_GENERIC", 0) || a.dtype != MN_DT_BF16 || (a.hd != 64 && a.hd != HD) || a.kv.block_size != BS ||
      a.Hkv <= 0 || a.H % a.Hkv != 0 || a.items == nullptr || a.row_splits == nullptr ||
      a.items_capacity < attention_items_capacity(a.B, a.M, a.H, a.Hkv))
    return false;
  if (a.hd == HD && (a.scratch == nullptr || a.scratch_bytes < attention_scratch_bytes(a.M, a.H, a.hd, a.max_ctx, a.dtype))) return false;
  const int ct = (a.H / a.Hkv * a.max_q + 15) / 16;
  if (a.hd == 64 || ct == 1) return ct <= 2;
  const int wgs = a.B * a.Hkv;
  return ct == 2 && a.append && pick_splits(a.max_ctx) == 1 && !MN_TUNE("MN_ATTN_NOFUSE", 0) && a.max_ctx <= KEYS_CT2_MAX_CTX &&
         wgs >= KEYS_CT2_MIN_WGS && wgs <= KEYS_CT2_MAX_WGS;
}
// Shape of the MFMA launch, from what the host knows (largest row count of a sequence, longest context).
struct MfmaShape {
  int ctw, nw, n_rg, n_splits, grid_items;
  bool keys;  // attn_keys_kernel
  bool list;  // the kernel takes its work from the list
};
static MfmaShape mfma_shape(const AttnArgs& a) {
  const int G = a.Hkv > 0 ? a.H / a.Hkv : 1;
  // the kernel covers NW * CTW column tiles of 16 stacked query rows per workgroup (4 waves with one or two tiles
  // each, or 5-6 waves with one tile each when that gives every wave the same work); longer stacks are cut into
  // row groups
  const int nt16_max = (G * a.max_q + 15) / 16;
  MfmaShape s;
  s.keys = keys_path(a);
  s.ctw = nt16_max <= 4 ? 1 : MAX_CT;
  s.nw = 4;
  if (s.keys) {
    s.ctw = nt16_max;
    s.nw = 1;  // (waves share the column tiles: a workgroup covers ctw of them)
    s.n_rg = 1;
  } else if ((nt16_max == 5 || nt16_max == 6) && MN_TUNE("MN_ATTN_NW", 0) != 4) { s.ctw = 1; s.nw = nt16_max; }
  s.n_rg = (nt16_max + s.nw * s.ctw - 1) / (s.nw * s.ctw);
  s.n_splits = a.hd == HD ? pick_splits(a.max_ctx) : 1;
  s.list = !(s.keys && s.n_splits == 1 && (long)a.B * a.Hkv <= KEYS_RESIDENT);
  const size_t bound = (size_t)a.B * s.n_rg * s.n_splits;
  s.grid_items = (int)(bound < a.items_capacity ? bound : a.items_capacity);
  return s;
}
static bool mfma_path(const AttnArgs& a) {
  // (the block-index staging of the longest context must fit the LDS beside the tile ring: about 390 000 tokens;
  // longer contexts take the generic kernel)
  return attention_mfma_supported(a.H, a.Hkv, a.hd, a.kv.block_size, a.dtype) && a.scratch != nullptr &&
         mfma_smem_bytes((a.max_ctx + KT - 1) / KT + 1) <= 160 * 1024 &&
         a.scratch_bytes >= attention_scratch_bytes(a.M, a.H, a.hd, a.max_ctx, a.dtype) && a.items != nullptr &&
         a.row_splits != nullptr &&
         a.items_capacity >= attention_items_capacity(a.B, a.M, a.H, a.Hkv);
}

AttnPlan attention_plan(const AttnArgs& a) {
  AttnPlan p{};
  if (a.M <= 0 || a.B <= 0 || !(keys_path(a) || mfma_path(a))) return p;
  const MfmaShape s = mfma_shape(a);
  if (!s.list) return p;
  p.items = a.items; p.row_splits = a.row_splits; p.grid_items = s.grid_items;
  p.tiles16_per_wg = s.nw * s.ctw; p.n_splits_max = s.n_splits;
  p.target_wgs = attention_target_workgroups(); p.min_tiles = attention_min_tiles();
  return p;
}

static void launch_merge(const AttnArgs& a, int n_splits, const float* o_part, const float* ml_part, hipStream_t st) {
  if (n_splits <= 1) return;
  attn_merge_kernel<<<(a.M * a.H + 7) / 8, 256, 0, st>>>(o_part, ml_part, n_splits, a.M, a.H, a.row_splits, reinterpret_cast<f16_t*>(a.out));
}

// A workgroup's waves split its keys: 8 waves up to one workgroup per CU, 4 (two workgroups per CU) beyond.  Measured with
// the append inside: 256 workgroups of 300-2000 keys 38.9 us with 8 waves (32.2 with its key loads as they are now), 42.0 with
// 4; 192 of 1024 keys 15.7 / 17.6; 320 of 512 keys 28.3 / 25.0.
template <int HDIM, int CT, int NW, bool FUSED>
static hipError_t launch_keys_nw(const AttnArgs& a, const MfmaShape& sh, float* o_part, float* ml_part, hipStream_t st) {
  constexpr size_t smem = (size_t)NW * 16 * (HDIM + 4) * sizeof(float);
  static std::once_flag attr_once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(attr_once, [] {
    attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(attn_keys_kernel<HDIM, CT, NW, FUSED>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  });
  if (attr_err != hipSuccess) return attr_err;
  attn_keys_kernel<HDIM, CT, NW, FUSED><<<(unsigned)a.Hkv * (unsigned)sh.grid_items, NW * 64, smem, st>>>(MN_ATTN_LEAD_OF(a), a, o_part, ml_part);
  return hipSuccess;
}
template <int HDIM, int CT>
static hipError_t launch_keys(const AttnArgs& a, const MfmaShape& sh, float* o_part, float* ml_part, hipStream_t st) {
  const int nw = MN_TUNE("MN_ATTN_KEYS_NW", 0);
  if (nw ? nw == 8 : a.B * a.Hkv <= 256)
    return a.qkv ? launch_keys_nw<HDIM, CT, 8, true>(a, sh, o_part, ml_part, st) : launch_keys_nw<HDIM, CT, 8, false>(a, sh, o_part, ml_part, st);
  return a.qkv ? launch_keys_nw<HDIM, CT, 4, true>(a, sh, o_part, ml_part, st) : launch_keys_nw<HDIM, CT, 4, false>(a, sh, o_part, ml_part, st);
}

bool attention_fuses_append(const AttnArgs& a) {
  if (a.M <= 0 || a.B <= 0 || MN_TUNE("MN_ATTN_NOFUSE", 0)) return false;
  if (a.dtype != MN_DT_BF16) return a.max_q <= GEN_NEW_ROWS;  // (attn_generic_kernel)
  return keys_path(a) && mfma_shape(a).n_splits == 1;
}

template <typename TA, typename T, bool FUSED>
static void launch_generic(const AttnArgs& a, hipStream_t st) {
  const dim3 grid(a.H, a.M);
  const bool wide = a.max_ctx > 256 && (long)a.M * a.H <= (a.max_ctx > GEN_LONG ? GEN_PAIRS : GEN_ALONE);
  const size_t smem = FUSED ? (size_t)2 * a.max_q * a.hd * sizeof(float) : 0;
  auto launch = [&](auto kernel, int threads) {
    kernel<<<grid, threads, smem, st>>>(a.rows.row_seq, a.rows.row_pos, a.rows.row_j, a.rows.row_slot, a.kv.block_tables, a.H, a.Hkv, a.hd, a.kv.block_size, a);
  };
  wide ? launch(attn_generic_kernel<TA, T, 1024, FUSED>, 1024) : launch(attn_generic_kernel<TA, T, 256, FUSED>, 256);
}

hipError_t launch_attention(const AttnArgs& a, hipStream_t st) {
  if (a.M <= 0 || a.B <= 0) return hipSuccess;
  if (keys_path(a)) {
    const MfmaShape sh = mfma_shape(a);
    AttnArgs k = a;
    if (!sh.list) k.items = nullptr;
    float* o_part = a.scratch;
    float* ml_part = a.scratch + (size_t)sh.n_splits * a.M * a.H * HD;
    hipError_t e;
    if (a.hd == 64) e = sh.ctw == 1 ? launch_keys<64, 1>(k, sh, o_part, ml_part, st) : launch_keys<64, 2>(k, sh, o_part, ml_part, st);
    else e = sh.ctw == 1 ? launch_keys<128, 1>(k, sh, o_part, ml_part, st) : launch_keys_nw<128, 2, 4, true>(k, sh, o_part, ml_part, st);
    if (e == hipSuccess) launch_merge(a, sh.n_splits, o_part, ml_part, st);
    return e;
  }
  if (mfma_path(a)) {
    const MfmaShape sh = mfma_shape(a);
    const int n_splits = sh.n_splits;
    float* o_part = a.scratch;
    float* ml_part = a.scratch + (size_t)n_splits * a.M * a.H * HD;
    // The block-index staging holds every block of the longest context: how many splits a sequence gets is
    // decided on the device from the whole batch (a large batch leaves even its longest sequence in one piece), so
    // a workgroup may have to walk all of a sequence's key tiles.  (Sized for the most splits instead, the array
    // was too short whenever the device chose fewer, and only the allocation granularity of the LDS covered it.)
    const int tiles_per_split = (a.max_ctx + KT - 1) / KT + 1;
    const size_t smem = mfma_smem_bytes(tiles_per_split);
    // once per process, whichever thread comes first; a refusal is returned by every call and nothing is launched
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [] {
      const void* fns[4] = {reinterpret_cast<const void*>(attn_mfma_kernel<1, 4>), reinterpret_cast<const void*>(attn_mfma_kernel<2, 4>),
                            reinterpret_cast<const void*>(attn_mfma_kernel<1, 5>), reinterpret_cast<const void*>(attn_mfma_kernel<1, 6>)};
      for (const void* f : fns) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) attr_err = e;
      }
    });
    if (attr_err != hipSuccess) return attr_err;
    const unsigned grid = (unsigned)a.Hkv * (unsigned)sh.grid_items;
    if (sh.nw == 5) attn_mfma_kernel<1, 5><<<grid, 320, smem, st>>>(MN_ATTN_LEAD_OF(a), a, o_part, ml_part);
    else if (sh.nw == 6) attn_mfma_kernel<1, 6><<<grid, 384, smem, st>>>(MN_ATTN_LEAD_OF(a), a, o_part, ml_part);
    else if (sh.ctw == 1) attn_mfma_kernel<1, 4><<<grid, 256, smem, st>>>(MN_ATTN_LEAD_OF(a), a, o_part, ml_part);
    else attn_mfma_kernel<2, 4><<<grid, 256, smem, st>>>(MN_ATTN_LEAD_OF(a), a, o_part, ml_part);
    launch_merge(a, n_splits, o_part, ml_part, st);
    return hipSuccess;
  }
  if (a.dtype == MN_DT_BF16) launch_generic<f16_t, f16_t, false>(a, st);
  else if (a.qkv) launch_generic<float, float, true>(a, st);
  else launch_generic<float, float, false>(a, st);
  return hipSuccess;
}

}  // namespace mn
