// Projections of small RMSNorm models (the drafting models), with the norms and the residual stream folded into them.
//
// A layer of such a model is a chain of launches that each hold a few hundred KB of weights: what it costs is the number of
// launches and the round trips inside one, not bytes.  Three things follow.
//  * A workgroup owns a few 16 x 16 output tiles over the whole of K: its waves take a k range each, ask for all of their
//    weights and activations at once (straight into the operand registers; there is nothing to share), and add up through LDS.
//    No partial sums go to memory.
//  * Because the sums are whole, the output projection and the second FFN projection update the residual stream themselves, and
//    the norm behind them needs no launch: RMSNorm is a factor per row, which the next projection applies to its sums.  The row
//    goes out as fp16(x * gain * s), s a power of two near 8 times the row's last 1 / rms, with the sum of squares of every
//    16 columns; the next projection adds those up while its loads are on their way.
//  * s is a guess, so the row's numbers are checked: a producer marks a tile (sign bit of its sum of squares) that left the fp16
//    range, and a consumer counts a row whose 1 / rms came out above s as marked.  A workgroup with marked rows does its sums again and
//    normalises those of them from fp32, exactly as norm_kernel does; a row's result does not depend on its neighbours' numbers.  Unmarked rows lose nothing against norm_kernel's fp16(x * gain / rms), whatever the
//    gains and however the row's energy is spread: the factor behind the sums is at most 1, so what is stored is no smaller than
//    what norm_kernel stores (no more of it is subnormal), and norm_kernel would not have saturated either.  (With s 2^9 times
//    smaller, gains of 2^-12 put the stored rows among the subnormals: the last layer's keys and values of a 256-wide model of two
//    layers were off by 6e-3, now by 4e-4 as with gains of 1.)
// Activations travel in operand order (common.h): with row-major ones a wave's fragment is 16 pieces of 64 bytes whose stride of
// K * 2 bytes puts them on few L2 channels (down projection of 95 rows 10.6 -> 7.5 us).
// Bound by launch and round trips: at 16 rows a launch takes 4.3 (QKV), 4.8 (output), 5.2 (gate||up) and 6.6 us (down, which
// brings 98 KB of weights and 98 KB of activations to each of 48 CUs); without any loads they take 3.9 to 4.4.  Per launch and
// layer of the 768-wide model before: norm 2 x 3.8, QKV and output 4.3, gate||up 6.2, down 4.6 us; at 95 rows 2 x 3.9, 6.5,
// 4.7, 9.9 and 7.0, then 5.1, 4.8, 8.4 and 7.8.
// A launch is one chain, so nothing in it may wait for what it does not need.  The compiler's code had three waits too many: for
// the sums of squares (or the residual row) before the weights were asked for, because loads of k-steps past the end were pending
// at the loop's back edge or the row stood behind a condition; for the first weights before the last were asked for; and for every
// second wave's sums in the LDS.  Without them and without a division per workgroup, 12 layers, whole passes: 16 rows at 16 keys
// 327 -> 310 us, at 1024 keys 434.6 -> 419.8; 95 rows 501.2 -> 493.6.
#include "launch.h"
#include "tune.h"
#include "../../include/minions_verify.h"

namespace mn {

constexpr int SMALL_MAX_D = 1024;             // widest model
constexpr float ROW_MARK = 65504.f;           // largest |x * s * gain|
constexpr float ROW_FACTOR_MAX = 1.f;         // largest rstd / s

__device__ __forceinline__ f16x8 norm8(const float* x, const float* gain, float rstd, bool& bad) {
  const f32x4 a = *reinterpret_cast<const f32x4*>(x), b = *reinterpret_cast<const f32x4*>(x + 4);
  const f32x4 ga = *reinterpret_cast<const f32x4*>(gain), gb = *reinterpret_cast<const f32x4*>(gain + 4);
  union { f16x8 v; uint32_t u[4]; } r;
  r.u[0] = pack2h_sat(a[0] * rstd * ga[0], a[1] * rstd * ga[1], bad);
  r.u[1] = pack2h_sat(a[2] * rstd * ga[2], a[3] * rstd * ga[3], bad);
  r.u[2] = pack2h_sat(b[0] * rstd * gb[0], b[1] * rstd * gb[1], bad);
  r.u[3] = pack2h_sat(b[2] * rstd * gb[2], b[3] * rstd * gb[3], bad);
  return r.v;
}

// CT x RT tiles of 16 columns x 16 rows per workgroup (HALF: 8 rows, each twice in the MFMA, whose other half is thrown away), NW waves
// along k, UF k-steps of 32 in flight per wave.
template <int CT, int RT, int NW, int UF, int MODE, bool HALF = false>
__global__ void __launch_bounds__(NW * 64, NW >= 16 ? 1 : 2) gemm_small_kernel(const void* a_, const void* w_, int M_, int N_, int K_, int ss_tiles_,
                                                                                 float* p0_, float* p1_, float* rstd_, SmallGemmArgs a) {
  a.a = a_; a.w = w_; a.M = M_; a.N = N_; a.K = K_; a.ss_tiles = ss_tiles_; a.rstd = rstd_;  // (launch.h: leading arguments)
  if (MODE == SMALL_RESIDUAL) { a.x = p0_; a.gain = p1_; }
  else { a.ss = p0_; a.inv_sc = p1_; }
  constexpr int NT = NW * 64, ROWS = HALF ? 8 : 16 * RT, TILES = CT * RT;
  constexpr bool TWO = NW * TILES > 48;      // the upper half of the waves hands its sums to the lower half first
  constexpr int NA = TWO ? NW / 2 : NW;
  constexpr int LP = 64 / ROWS;              // lanes of a wave that share a row's sums of squares
  __shared__ f32x4 s_acc[NA][TILES][64];
  __shared__ float s_part[NW][ROWS];
  static_assert(TILES * 64 <= NT || MODE != SMALL_RESIDUAL, "one piece per thread");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, g = lane >> 4;
  // id -> (column group, row group): the row groups of a column group on one XCD, whose L2 then holds its weights once
  // (ids are dealt to the XCDs in turn, x first)
  const int groups = ((a.N + 15) / 16 + CT - 1) / CT, cg = (int)blockIdx.z * 8 + (int)blockIdx.x, rg = blockIdx.y;
  if (cg >= groups) return;  // (whole workgroup: padding of the grid)
  const int t0 = cg * CT, m0 = rg * ROWS;
  const bool scaled = MODE != SMALL_RESIDUAL && a.ss != nullptr;

  // sums of squares of the rows: a strided share per wave and LP-th of its lanes, asked for first and looked at behind the products
  constexpr int SHARES = NW * LP, SS = (SMALL_MAX_D / 16 + SHARES - 1) / SHARES;
  const int share = wave * LP + min(lane / ROWS, LP - 1);
  float ss_v[SS], inv_sc = 1.f;
  if (scaled) {
    const int m = min(m0 + lane % ROWS, a.M - 1);
    inv_sc = a.inv_sc[m];
#pragma unroll
    for (int u = 0; u < SS; ++u) ss_v[u] = a.ss[(size_t)min(share + u * SHARES, a.ss_tiles - 1) * a.M + m];
  }
  // the residual stream's old values and the next norm's gains (each thread owns one piece of four columns of a row; the others
  // ask for one as well: behind a condition the loads would be waited for before the weights are asked for)
  const int pt = min(wave, TILES - 1);       // tile = ct * RT + rt
  const int pm = m0 + pt % RT * 16 + (HALF ? l16 & 7 : l16), pn = (t0 + pt / RT) * 16 + 4 * g;
  f32x4 x_old, gain;
  float rs_old;
  const bool piece = MODE == SMALL_RESIDUAL && tid < TILES * 64 && pm < a.M && pn < a.N && !(HALF && l16 >= 8);
  if (MODE == SMALL_RESIDUAL) {
    const int cm = min(pm, a.M - 1), cn = min(pn, a.N - 4);
    x_old = *reinterpret_cast<const f32x4*>(a.x + (size_t)cm * a.N + cn);
    gain = *reinterpret_cast<const f32x4*>(a.gain + cn);
    rs_old = a.rstd[cm];
  }

  const int ks_all = a.K / KSTEP, per = (ks_all + NW - 1) / NW;
  const int k0 = min(wave * per, ks_all), k1 = min(k0 + per, ks_all);
  const f16_t* A = reinterpret_cast<const f16_t*>(a.a);
  const uint16_t* W = reinterpret_cast<const uint16_t*>(a.w);
  // (rows past the last one repeat it: they feed outputs that are never stored)
  const f16_t* a_tile[RT];
  int a_step[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    const int t = min(m0 / 16 + r, (a.M - 1) / 16), rows = min(16, a.M - 16 * t);
    a_step[r] = 32 * rows;
    a_tile[r] = A + (size_t)t * 16 * a.K + (g * rows + min(HALF ? (m0 & 8) + (l16 & 7) : l16, rows - 1)) * 8;
  }
  bool bad = false;
  float rstd = 0.f, f = 1.f;                 // of row m0 + lane (lanes below ROWS)
  bool renorm = false;
  auto sums = [&](auto slow_c) {
    constexpr bool SLOW = decltype(slow_c)::value;
    constexpr int U = SLOW ? 1 : UF;
    f32x4 acc[CT][RT];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[c][r] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int kk = k0; kk < k1; kk += U) {
      u32x4 wf[U][CT];
      f16x8 af[U][RT];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = min(kk + u, k1 - 1);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          const int t = t0 + c;              // (an odd last tile of a group lies inside the padded matrix)
          wf[u][c] = *reinterpret_cast<const u32x4*>(W + ((size_t)(t >> 3) * (a.K / KB) + (k >> 2)) * WBLOCK + ((t & 7) * KS + (k & 3)) * 512 + lane * 8);
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          af[u][r] = *reinterpret_cast<const f16x8*>(a_tile[r] + (size_t)k * a_step[r]);
          if constexpr (SLOW) {              // (the rows beside a marked one keep their operands and with them every bit)
            const float rs = __shfl(rstd, r * 16 + l16, 64);
            if (__shfl((int)renorm, r * 16 + l16, 64))
              af[u][r] = norm8(a.x + (size_t)min(m0 + r * 16 + l16, a.M - 1) * a.K + k * KSTEP + g * 8, a.gain + k * KSTEP + g * 8, rs, bad);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);     // (every load goes out before the first product)
      if constexpr (!SLOW)                   // (and the arguments that the end needs are fetched meanwhile)
        asm volatile("" ::"s"(a.out), "s"(a.inv_d), "s"(a.eps), "s"(a.dev_status), "s"(a.x), "s"(a.gain), "s"(a.ss), "s"(a.inv_sc));
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (kk + u >= k1) break;             // (wave-uniform)
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
          for (int r = 0; r < RT; ++r) acc[c][r] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, wf[u][c]), af[u][r], acc[c][r], 0, 0, 0);
      }
      // (vmcnt(0): loads of k-steps past the end, pending at the back edge, would make the first pass wait for the sums of
      // squares before it asks for its weights)
      __builtin_amdgcn_s_waitcnt((7 << 4) | (15 << 8));
    }
    if constexpr (TWO) {
      if (wave >= NA) {
#pragma unroll
        for (int t = 0; t < TILES; ++t) s_acc[wave - NA][t][lane] = acc[t / RT][t % RT];
      }
      __syncthreads();
      if (wave < NA) {
#pragma unroll
        for (int t = 0; t < TILES; ++t) s_acc[wave][t][lane] = acc[t / RT][t % RT] + s_acc[wave][t][lane];
      }
    } else {
#pragma unroll
      for (int t = 0; t < TILES; ++t) s_acc[wave][t][lane] = acc[t / RT][t % RT];
    }
  };
  sums(BoolC<false>{});
  if (scaled) {
    float sq = 0.f;
    uint32_t mark = 0;
#pragma unroll
    for (int u = 0; u < SS; ++u)
      if (share + u * SHARES < a.ss_tiles) {
        sq += __builtin_fabsf(ss_v[u]);
        mark |= __float_as_uint(ss_v[u]);
      }
    uint32_t x, y;
    if (LP == 4) {
      lane_pair<16>(__float_as_uint(sq), x, y);
      sq = __uint_as_float(x) + __uint_as_float(y);
      lane_pair<16>(mark, x, y);
      mark = x | y;
    }
    if (LP >= 2) {
      lane_pair<32>(__float_as_uint(sq), x, y);
      sq = __uint_as_float(x) + __uint_as_float(y);
      lane_pair<32>(mark, x, y);
      mark = x | y;
    }
    // (the mark travels in the sign)
    if (lane < ROWS) s_part[wave][lane] = __uint_as_float((__float_as_uint(sq) & 0x7fffffffu) | (mark & 0x80000000u));
  }
  __syncthreads();
  if (scaled) {                              // (every wave for itself: all see all rows)
    float t = 0.f;
    uint32_t mark = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float v = s_part[w][lane % ROWS];
      t += __builtin_fabsf(v);
      mark |= __float_as_uint(v);
    }
    rstd = 1.f / sqrtf(t * a.inv_d + a.eps);
    f = rstd * inv_sc;
    if (cg == 0 && tid < ROWS && m0 + tid < a.M) a.rstd[m0 + tid] = rstd;
    renorm = mark >> 31 || !(f <= ROW_FACTOR_MAX);
    if (__any((int)renorm)) {                // (the same in every wave)
      __syncthreads();
      sums(BoolC<true>{});
      __syncthreads();
      if (renorm) f = 1.f;
    }
  }

  // lane holds D[n = 4g + i][m = l16] of a tile; the waves' sums are added in wave order
  auto total = [&](int tile, int ln) {
    f32x4 p[NA];
#pragma unroll
    for (int w = 0; w < NA; ++w) p[w] = s_acc[w][tile][ln];
    __builtin_amdgcn_sched_barrier(0);       // (one round trip to the LDS, not one for every second wave)
    f32x4 v = p[0];
#pragma unroll
    for (int w = 1; w < NA; ++w) v += p[w];
    return v;
  };
  if constexpr (MODE == SMALL_OUT) {
    for (int i = tid; i < TILES * 64; i += NT) {          // (whole waves)
      const int tile = i >> 6, r = tile % RT * 16 + (i & 15), m = m0 + r, n = (t0 + tile / RT) * 16 + ((i >> 4) & 3) * 4;
      f32x4 v = total(tile, i & 63);
      if (scaled) v *= __shfl(f, r, 64);
      if (m < a.M && n < a.N) *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.out) + (size_t)m * a.N + n) = v;
    }
  } else if constexpr (MODE == SMALL_SWIGLU) {
    static_assert(MODE != SMALL_SWIGLU || CT % 2 == 0, "gate and up tiles alternate");
    for (int i = tid; i < RT * (CT / 2) * 64; i += NT) {  // (whole waves)
      const int pr = (i >> 6) / RT, rt = (i >> 6) % RT;
      const int r = rt * 16 + (i & 15), m = m0 + r, c = (t0 / 2 + pr) * 16 + ((i >> 4) & 3) * 4;
      f32x4 gt = total(2 * pr * RT + rt, i & 63), up = total((2 * pr + 1) * RT + rt, i & 63);
      if (scaled) { const float fr = __shfl(f, r, 64); gt *= fr; up *= fr; }
      float o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = gt[e] / (1.f + __expf(-gt[e])) * up[e];
      if (m < a.M && c < (a.N >> 1))
        *reinterpret_cast<uint2*>(reinterpret_cast<f16_t*>(a.out) + operand_at(m, c, a.M, a.N >> 1)) = make_uint2(pack2h_sat(o[0], o[1], bad), pack2h_sat(o[2], o[3], bad));
    }
  } else {
    if (tid < TILES * 64) {                  // (whole waves)
      f32x4 v = x_old + total(tid >> 6, lane);
      // 2^3 times the power of two at or below the row's last 1 / rms (positive and finite: eps > 0 or a row of zeros): the row
      // may shrink to a quarter of its rms before it is marked, or grow until an element is 8188 times the rms before
      const float s = __uint_as_float(min(max(__float_as_uint(rs_old) & 0x7f800000u, 0x08000000u), 0x75000000u) + 0x01800000u);
      f32x4 h = v * s * gain;
      bool over = false;
      float q = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        over |= !(__builtin_fabsf(h[e]) <= ROW_MARK);
        h[e] = __builtin_fminf(__builtin_fmaxf(h[e], -ROW_MARK), ROW_MARK);
        q += v[e] * v[e];
      }
      uint32_t o = over, y0, y1;
      lane_pair<16>(__float_as_uint(q), y0, y1);
      q = __uint_as_float(y0) + __uint_as_float(y1);
      lane_pair<32>(__float_as_uint(q), y0, y1);
      q = __uint_as_float(y0) + __uint_as_float(y1);
      lane_pair<16>(o, y0, y1);
      o = y0 | y1;
      lane_pair<32>(o, y0, y1);
      o = y0 | y1;
      if (piece) {
        *reinterpret_cast<f32x4*>(a.x + (size_t)pm * a.N + pn) = v;
        *reinterpret_cast<uint2*>(reinterpret_cast<f16_t*>(a.out) + operand_at(pm, pn, a.M, a.N)) = make_uint2(pack2h(h[0], h[1]), pack2h(h[2], h[3]));
        if (g == 0) {
          a.ss[(size_t)(pn >> 4) * a.M + pm] = __uint_as_float((__float_as_uint(q) & 0x7fffffffu) | (o ? 0x80000000u : 0u));
          if (pn == 0) a.inv_sc[pm] = 1.f / s;  // (exact)
        }
      }
    }
  }
  if (bad && a.dev_status) atomicOr(a.dev_status, MN_DEV_RANGE);
}

template <int CT, int RT, int NW, int UF, int MODE, bool HALF = false>
static void launch_small_u(const SmallGemmArgs& a, hipStream_t st) {
  constexpr int ROWS = HALF ? 8 : 16 * RT;
  const int groups = ((a.N + 15) / 16 + CT - 1) / CT, rgs = (a.M + ROWS - 1) / ROWS;
  gemm_small_kernel<CT, RT, NW, UF, MODE, HALF><<<dim3(8, rgs, (groups + 7) / 8), NW * 64, 0, st>>>(
      a.a, a.w, a.M, a.N, a.K, a.ss_tiles, MODE == SMALL_RESIDUAL ? a.x : a.ss, MODE == SMALL_RESIDUAL ? const_cast<float*>(a.gain) : a.inv_sc, a.rstd, a);
}
// Waves and k-steps in flight, so that every wave asks for its whole k range at once: eight waves of three k-steps for K up to 768, of four
// beyond; where the residual stream wants whole sums of a long K, 16 waves of six up to 3072 and of eight beyond.  With three and six
// only, models wider than 768 made two round trips of every launch: six layers, 1024 wide, FFN 3584, weights in the caches and not, 1 row
// 191 -> 179 us and 240 -> 229, 16 rows 196 -> 185 and 245 -> 237, 64 rows 238 -> 230 and 299 -> 294; FFN 3968 1 row 199 -> 186 and 252 -> 237.
template <int CT, int RT, int MODE, bool HALF = false>
static void launch_small(const SmallGemmArgs& a, hipStream_t st) {
  if constexpr (MODE == SMALL_RESIDUAL) {
    if (a.K <= 8 * 3 * KSTEP) launch_small_u<CT, RT, 8, 3, MODE, HALF>(a, st);
    else if (a.K <= 16 * 6 * KSTEP) launch_small_u<CT, RT, 16, 6, MODE, HALF>(a, st);
    else launch_small_u<CT, RT, 16, 8, MODE, HALF>(a, st);
  } else {
    if (a.K <= 8 * 3 * KSTEP) launch_small_u<CT, RT, 8, 3, MODE, HALF>(a, st);
    else launch_small_u<CT, RT, 8, 4, MODE, HALF>(a, st);
  }
}

// Rows up to which a model whose matrices are all small (gemm.hip) takes these kernels.  Every row group reads the weights again
// and every column group the rows, so the launches saved lose against tiles of 160 rows and more at some point; 12 layers, whole
// passes before and now: 768 wide 16 rows 570 and 518 us, 96 rows 613 and 490, 112 1061 and 550, 216 1577 and 703, 528 1691 and
// 1127, 816 1839 and 1553, 1344 2014 and 2240; 1024 wide (FFN 3968) 16 567 and 550, 96 681 and 617, 640 2061 and 1930, 816 2188
// and 2566; 512 wide 16 384 and 314, 400 1057 and 559.
constexpr int SMALL_MAX_ROWS = 640;
bool gemm_small_model(int M, int n_qkv, int d_model, int hdim, int w1_rows, int d_ffn) {
  return M <= MN_TUNE("MN_SMALL_ROWS", SMALL_MAX_ROWS) && d_model <= SMALL_MAX_D && gemm_small_matrix(n_qkv, d_model) && gemm_small_matrix(d_model, hdim) && gemm_small_matrix(w1_rows, d_model) &&
         gemm_small_matrix(d_model, d_ffn);
}

// Tiles per workgroup.  95 rows, microseconds: QKV 1 x 3 tiles (columns x rows) 7.0, 1 x 2 6.0, 2 x 3 6.5, 2 x 2 5.7, 2 x 1 6.2;
// gate||up 2 x 3 9.2, 2 x 2 9.8, 2 x 1 11.6, 4 x 3 9.1; residual 1 x 1 and 1 x 2 alike, 1 x 3 10.8 (spills).  At 33 to 48 rows, one
// row group of three tiles, 4 x 3 would leave gate||up to half as many CUs as 2 x 3: passes of six layers, weights in the caches and not, 48
// rows, 768 wide 191 -> 184 us and 242 -> 233, 1024 wide 223 -> 217 and 285 -> 275; at 64 rows 1024 wide 2 x 3 is slower, 237 and 230.  From 9 to 32 rows the residual kernels take 8 rows per workgroup: as many weights, half the activations for
// each of twice the CUs (16 rows, K = 3072: 6.6 -> 6.0 us; whole passes at 16, 24 and 32 rows 465 -> 455, 512 -> 486, 544 -> 512; at 48 no
// change, at 96 490 -> 523).  QKV at 17 to 32 rows 2 x 2 tiles -> 1 x 1: 1 % of the pass; gate||up 2 x 2 -> 2 x 1 2 % slower.  4 waves with six k-steps each are no faster than 8 with three.
void launch_gemm_small(const SmallGemmArgs& a, int mode, hipStream_t st) {
  const int tiles = (a.M + 15) / 16;
  if (mode == SMALL_OUT) {
    if (tiles <= 2) launch_small<1, 1, SMALL_OUT>(a, st);
    else launch_small<2, 2, SMALL_OUT>(a, st);
  } else if (mode == SMALL_SWIGLU) {
    if (tiles == 1) launch_small<2, 1, SMALL_SWIGLU>(a, st);
    else if (tiles == 2) launch_small<2, 2, SMALL_SWIGLU>(a, st);
    else if (tiles == 3) launch_small<2, 3, SMALL_SWIGLU>(a, st);
    else launch_small<4, 3, SMALL_SWIGLU>(a, st);
  } else {
    if (a.M > 8 && tiles <= 2) launch_small<1, 1, SMALL_RESIDUAL, true>(a, st);
    else if (tiles == 1) launch_small<1, 1, SMALL_RESIDUAL>(a, st);
    else launch_small<1, 2, SMALL_RESIDUAL>(a, st);
  }
}

}  // namespace mn
