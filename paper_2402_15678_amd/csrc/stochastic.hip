// Stochastic verification (paper section 2.1, the general rule; longest-prefix acceptance on argmax
// tokens is its temperature -> 0 case).  For every scored position the kernel decides whether the
// speculated token survives (kept outright when the SSM's probability q does not exceed the LLM's o,
// otherwise rejected with probability 1 - o/q) and, where it does not, or at the position after the
// last speculated token, draws a token from max(0, o - q) renormalised (from o itself after the last
// one).  The result has the layout of the greedy token array, with a surviving position holding its
// own speculated token, so the same acceptance and commit kernel turns it into the step's output:
// the first position whose entry differs from the speculated token is the first rejection.
//
// Arithmetic: fp64 throughout (the scores arrive as fp32).  A decision compares a 53-bit uniform
// number with a ratio or a running sum known to about 1e-14 relative, so it is reproducible by any
// other fp64 evaluation of the same definition except on a set of measure ~1e-14.
// Random numbers: Philox-4x32 with 10 rounds (Salmon et al., SC 2011), key = seed, counter =
// (sequence, position, step + consumer tag): a position's numbers do not depend on the batch it is scored in.
//
// The same file holds the drafting side of the rule: draft_sample_kernel draws an SSM's next token from
// its own q = softmax(scores / T) and writes q out for the verifier.
#include "launch.h"
#include "../../include/minions_verify.h"

namespace mn {

__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t hi0 = __umulhi(0xD2511F53u, c[0]), lo0 = 0xD2511F53u * c[0];
    const uint32_t hi1 = __umulhi(0xCD9E8D57u, c[2]), lo1 = 0xCD9E8D57u * c[2];
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

// 27 + 26 random bits -> [0, 1)
__device__ __forceinline__ double unit_double(uint32_t hi, uint32_t lo) {
  return ((double)(hi >> 5) * 67108864.0 + (double)(lo >> 6)) * (1.0 / 9007199254740992.0);
}

// One workgroup of 16 waves per row, the row's exponentials in registers.  The kernels are bound by the fp64
// exponentials of one row on one CU (about 25 fp64 instructions per token, 64 lanes per clock: 6 us for 32000 tokens) and by
// the chain load -> maximum -> exponentials -> sum -> draw, so a row is read once, every exponential is computed once,
// and every sum is a wave reduction.  Measured at 32000 tokens: 21.9 us for the 144 positions of 16 requests and 16.8 us
// for 16 drafted tokens; 149 and 162 us with 256 threads per row, the scores re-read for every pass and one thread
// adding the 256 partial sums of every tile.
constexpr int SV_THREADS = 1024;
constexpr int SV_WAVES = SV_THREADS / 64;
constexpr int SV_BLOCK = 256;                         // tokens a wave takes at once: lane l holds 4l .. 4l+3 of them
constexpr int SV_TILE = SV_WAVES * SV_BLOCK;          // tokens the workgroup takes at once
constexpr int SV_REG_TILES = 8;                       // rows of up to 32768 tokens stay in registers (8 doubles x 4 per
                                                      // thread: 64 of the 128 registers 16 waves leave each other)
constexpr int SV_MAX_SEGS = 1024;
constexpr int SV_MAX_VOCAB = 1 << 21;

// Token order.  The row is cut into segments of `grp` consecutive blocks of 256 tokens; segment s belongs to wave s % 16,
// so (segment, block, lane, element) is token order.  grp = 1 up to 262144 tokens; larger rows take longer
// segments, so that their sums fit the shared array.
__device__ __forceinline__ int seg_blocks(int V) { return (V + SV_MAX_SEGS * SV_BLOCK - 1) / (SV_MAX_SEGS * SV_BLOCK); }

// (rows start at any multiple of 4 bytes: the vocabulary need not be a multiple of 4)
// four consecutive values of a row, `pad` past its end
__device__ __forceinline__ f32x4 load_row4(const float* __restrict__ R, int v, int V, float pad) {
  if (v + 3 < V) {
    const f32x4_u x = *reinterpret_cast<const f32x4_u*>(R + v);
    return (f32x4){x[0], x[1], x[2], x[3]};
  }
  f32x4 r = {pad, pad, pad, pad};
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (v + e < V) r[e] = R[v + e];
  return r;
}

// (see wave_reduce)
template <typename F>
__device__ __forceinline__ double both_halves(double v, F f) {
  return __hiloint2double((int)f((uint32_t)__double2hiint(v)), (int)f((uint32_t)__double2loint(v)));
}
template <int STEP>
__device__ __forceinline__ double lane_swap_d(double v) {
  return both_halves(v, [](uint32_t x) { return lane_swap<STEP>(x); });
}
// x and y hold values of lanes; afterwards a lane's sum is that of its x (lower half of the pair) or y (upper half) and the same
// of the lane DIST away
template <int DIST>
__device__ __forceinline__ double lane_halve_d(double x, double y) {
  const uint32_t xl = (uint32_t)__double2loint(x), yl = (uint32_t)__double2loint(y), xh = (uint32_t)__double2hiint(x), yh = (uint32_t)__double2hiint(y);
  const auto l = DIST == 16 ? __builtin_amdgcn_permlane16_swap(xl, yl, false, false) : __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
  const auto h = DIST == 16 ? __builtin_amdgcn_permlane16_swap(xh, yh, false, false) : __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
  return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
}
__device__ __forceinline__ double wave_sum_d(double v) {
  v += lane_swap_d<LANE_1>(v);
  v += lane_swap_d<LANE_2>(v);
  v += lane_swap_d<LANE_4>(v);
  v += lane_swap_d<LANE_8>(v);
  v = lane_halve_d<16>(v, v);
  return lane_halve_d<32>(v, v);
}

// one double from another lane by DPP, 0 where there is none or the row (of 16 lanes) is not in ROWS
template <int CTRL, int ROWS>
__device__ __forceinline__ double lane_get_d(double v) {
  return both_halves(v, [](uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false); });
}
// inclusive prefix sums over the lanes (row_shr 1, 2, 4, 8, then the last lane of row 0 and 2 to the next row, of row 1 to 2 and 3)
__device__ __forceinline__ double wave_scan_d(double v) {
  v += lane_get_d<0x111, 0xf>(v);
  v += lane_get_d<0x112, 0xf>(v);
  v += lane_get_d<0x114, 0xf>(v);
  v += lane_get_d<0x118, 0xf>(v);
  v += lane_get_d<0x142, 0xa>(v);
  v += lane_get_d<0x143, 0xc>(v);
  return v;
}
__device__ __forceinline__ double lane_before_d(double v) { return lane_get_d<0x138, 0xf>(v); }  // wave_shr:1; 0 in lane 0
__device__ __forceinline__ double lane_63_d(double v) {
  return both_halves(v, [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, 63); });
}

struct DrawShared {
  double seg[SV_MAX_SEGS];    // mass of every segment
  double2 pow2[64];           // 2^(j/64), rest
  double red[SV_WAVES];
  float redf[SV_WAVES];
  double target[2];           // target inside the chosen segment, total mass
  int pick[2];                // chosen segment, chosen token
};

// a * b + c with c in scalar registers.  (The compiler's choice is the two-address form with the constant copied to vector
// registers first, three instructions for one.)
__device__ __forceinline__ double fma_vvs(double a, double b, double c) {
  double r;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
  return r;
}

// x / c for a divisor that is the same for the whole row, inv = 1 / c: one correction step makes the product the
// rounded quotient.  (c and inv normal numbers, x finite: the caller sees to both)
__device__ __forceinline__ double div_by(double x, double c, double inv) {
  const double q = x * inv;
  return fma(fma(-c, q, x), inv, q);
}

// 2^(j/64), j = 0 .. 63, each as its nearest double and what that leaves over
__device__ const double kPow2[128] = {
    0x1.0000000000000p+0, 0x0.0p+0, 0x1.02c9a3e778061p+0, -0x1.19083535b085dp-56,
    0x1.059b0d3158574p+0, 0x1.d73e2a475b465p-55, 0x1.0874518759bc8p+0, 0x1.186be4bb284ffp-57,
    0x1.0b5586cf9890fp+0, 0x1.8a62e4adc610bp-54, 0x1.0e3ec32d3d1a2p+0, 0x1.03a1727c57b53p-59,
    0x1.11301d0125b51p+0, -0x1.6c51039449b3ap-54, 0x1.1429aaea92de0p+0, -0x1.32fbf9af1369ep-54,
    0x1.172b83c7d517bp+0, -0x1.19041b9d78a76p-55, 0x1.1a35beb6fcb75p+0, 0x1.e5b4c7b4968e4p-55,
    0x1.1d4873168b9aap+0, 0x1.e016e00a2643cp-54, 0x1.2063b88628cd6p+0, 0x1.dc775814a8495p-55,
    0x1.2387a6e756238p+0, 0x1.9b07eb6c70573p-54, 0x1.26b4565e27cddp+0, 0x1.2bd339940e9d9p-55,
    0x1.29e9df51fdee1p+0, 0x1.612e8afad1255p-55, 0x1.2d285a6e4030bp+0, 0x1.0024754db41d5p-54,
    0x1.306fe0a31b715p+0, 0x1.6f46ad23182e4p-55, 0x1.33c08b26416ffp+0, 0x1.32721843659a6p-54,
    0x1.371a7373aa9cbp+0, -0x1.63aeabf42eae2p-54, 0x1.3a7db34e59ff7p+0, -0x1.5e436d661f5e3p-56,
    0x1.3dea64c123422p+0, 0x1.ada0911f09ebcp-55, 0x1.4160a21f72e2ap+0, -0x1.ef3691c309278p-58,
    0x1.44e086061892dp+0, 0x1.89b7a04ef80d0p-59, 0x1.486a2b5c13cd0p+0, 0x1.3c1a3b69062f0p-56,
    0x1.4bfdad5362a27p+0, 0x1.d4397afec42e2p-56, 0x1.4f9b2769d2ca7p+0, -0x1.4b309d25957e3p-54,
    0x1.5342b569d4f82p+0, -0x1.07abe1db13cadp-55, 0x1.56f4736b527dap+0, 0x1.9bb2c011d93adp-54,
    0x1.5ab07dd485429p+0, 0x1.6324c054647adp-54, 0x1.5e76f15ad2148p+0, 0x1.ba6f93080e65ep-54,
    0x1.6247eb03a5585p+0, -0x1.383c17e40b497p-54, 0x1.6623882552225p+0, -0x1.bb60987591c34p-54,
    0x1.6a09e667f3bcdp+0, -0x1.bdd3413b26456p-54, 0x1.6dfb23c651a2fp+0, -0x1.bbe3a683c88abp-57,
    0x1.71f75e8ec5f74p+0, -0x1.16e4786887a99p-55, 0x1.75feb564267c9p+0, -0x1.0245957316dd3p-54,
    0x1.7a11473eb0187p+0, -0x1.41577ee04992fp-55, 0x1.7e2f336cf4e62p+0, 0x1.05d02ba15797ep-56,
    0x1.82589994cce13p+0, -0x1.d4c1dd41532d8p-54, 0x1.868d99b4492edp+0, -0x1.fc6f89bd4f6bap-54,
    0x1.8ace5422aa0dbp+0, 0x1.6e9f156864b27p-54, 0x1.8f1ae99157736p+0, 0x1.5cc13a2e3976cp-55,
    0x1.93737b0cdc5e5p+0, -0x1.75fc781b57ebcp-57, 0x1.97d829fde4e50p+0, -0x1.d185b7c1b85d1p-54,
    0x1.9c49182a3f090p+0, 0x1.c7c46b071f2bep-56, 0x1.a0c667b5de565p+0, -0x1.359495d1cd533p-54,
    0x1.a5503b23e255dp+0, -0x1.d2f6edb8d41e1p-54, 0x1.a9e6b5579fdbfp+0, 0x1.0fac90ef7fd31p-54,
    0x1.ae89f995ad3adp+0, 0x1.7a1cd345dcc81p-54, 0x1.b33a2b84f15fbp+0, -0x1.2805e3084d708p-57,
    0x1.b7f76f2fb5e47p+0, -0x1.5584f7e54ac3bp-56, 0x1.bcc1e904bc1d2p+0, 0x1.23dd07a2d9e84p-55,
    0x1.c199bdd85529cp+0, 0x1.11065895048ddp-55, 0x1.c67f12e57d14bp+0, 0x1.2884dff483cadp-54,
    0x1.cb720dcef9069p+0, 0x1.503cbd1e949dbp-56, 0x1.d072d4a07897cp+0, -0x1.cbc3743797a9cp-54,
    0x1.d5818dcfba487p+0, 0x1.2ed02d75b3707p-55, 0x1.da9e603db3285p+0, 0x1.c2300696db532p-54,
    0x1.dfc97337b9b5fp+0, -0x1.1a5cd4f184b5cp-54, 0x1.e502ee78b3ff6p+0, 0x1.39e8980a9cc8fp-55,
    0x1.ea4afa2a490dap+0, -0x1.e9c23179c2893p-54, 0x1.efa1bee615a27p+0, 0x1.dc7f486a4b6b0p-54,
    0x1.f50765b6e4540p+0, 0x1.9d3e12dd8a18bp-54, 0x1.fa7c1819e90d8p+0, 0x1.74853f3a5931ep-55,
};

// exp((l - max) / T), table-driven (P. T. P. Tang, ACM TOMS 15(2), 1989): (l - max) / T = n ln2/64 + r with |r| <= ln2/128, and
// exp = 2^(n >> 6) * 2^((n & 63)/64) * (1 + r + .. + r^5/120), the sixth-order term below 2^-54.  The 64 powers lie in LDS, in
// two pieces (their rounding would be the largest error).  Relative error against 64-bit mantissas, 400000 arguments
// in [-20, 0]: rms 4.8e-17, largest 1.4e-16 (a correctly rounded exponential: 4.7e-17 and 1.1e-16).
// About half the instructions of the general function (arguments are never positive), which is most of these kernels' time.
// The quotient is not rounded on its own: r comes out of one fma with T's reciprocal, so its error is the reciprocal's
// rounding, what a rounded quotient's would be.  For temperatures so extreme that the reciprocal leaves the normal
// range (inv == 0) the general function and a division.  Differences below -800 T are cut there (the exponential is zero long
// before), so that a masked token (minus infinity) stays finite; NaN passes through.  The cut is on the fp64 difference: 800 T
// may be far below the spacing of the scores in fp32, and the largest score may be the type's lowest value.
struct Temp {
  double T, inv, per_step;   // 1 / T, 64 / (T ln2)
  const double2* pow2;       // [64] 2^(j/64), rest
  double dmx;                // largest score of the row
  double lowest;             // -800 T
  double sixth_order;        // 1 / 120 (in vector registers: an instruction reads one scalar constant)
  float near;                // scores from here on are within 690 T of the largest (see mass4); NaN or more than any score: none are
  __device__ __forceinline__ void largest(float mx) {
    dmx = (double)mx;
    near = inv == 0.0 ? INFINITY : __double2float_ru(dmx - 690.0 * T);
  }
  // N exponentials side by side (one is a chain of fifteen dependent operations and an LDS read).  SMALL: a result may be below the
  // normal range, an argument below the cut or not a number.
  template <bool SMALL, int N>
  __device__ __forceinline__ void table_exp(const float (&l)[N], double (&m)[N]) const {
    double d[N], t[N], nd[N], r[N], p[N], sq[N];
    double2 c[N];
    int n[N];
#pragma unroll
    for (int e = 0; e < N; ++e) {
      d[e] = (double)l[e] - dmx;
      if (SMALL) d[e] = d[e] < lowest ? lowest : d[e];
    }
#pragma unroll
    for (int e = 0; e < N; ++e) t[e] = fma_vvs(d[e], per_step, 6755399441055744.0);  // 1.5 * 2^52: the nearest whole number sits in the low bits
#pragma unroll
    for (int e = 0; e < N; ++e) n[e] = (int)(uint32_t)__double_as_longlong(t[e]);
#pragma unroll
    for (int e = 0; e < N; ++e) c[e] = pow2[n[e] & 63];
#pragma unroll
    for (int e = 0; e < N; ++e) nd[e] = t[e] - 6755399441055744.0;
#pragma unroll
    for (int e = 0; e < N; ++e) r[e] = fma(d[e], inv, nd[e] * -0x1.62e42fefap-7);  // ln2/64, its first 33 bits (the product with n is exact) ...
#pragma unroll
    for (int e = 0; e < N; ++e) r[e] = fma(nd[e], -0x1.cf79abc9e3b3ap-46, r[e]);   // ... and the rest
#pragma unroll
    for (int e = 0; e < N; ++e) p[e] = fma_vvs(r[e], sixth_order, 1.0 / 24.0);
#pragma unroll
    for (int e = 0; e < N; ++e) sq[e] = r[e] * r[e];
#pragma unroll
    for (int e = 0; e < N; ++e) p[e] = fma_vvs(r[e], p[e], 1.0 / 6.0);
#pragma unroll
    for (int e = 0; e < N; ++e) p[e] = fma(r[e], p[e], 0.5);
#pragma unroll
    for (int e = 0; e < N; ++e) p[e] = fma(sq[e], p[e], r[e]);
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const double y = c[e].x + fma(c[e].x, p[e], c[e].y);
      m[e] = SMALL ? ldexp(y, n[e] >> 6) : __hiloint2double(__double2hiint(y) + ((n[e] & ~63) << 14), __double2loint(y));
    }
  }
  __device__ __forceinline__ double mass(float l) const {
    if (inv == 0.0) return exp(((double)l - dmx) / T);  // (uniform)
    const float one[1] = {l};
    double m[1];
    table_exp<true, 1>(one, m);
    return m[0];
  }
  // The masses of four scores, bit for bit those of mass().  Where every score of the wave is within 690 T of the largest the
  // powers of two are added to the exponent field and nothing is cut: the comparison, the selections and the ldexp were a quarter
  // of these kernels' arithmetic.
  __device__ __forceinline__ void mass4(const f32x4& l, double (&m)[4]) const {
    const float x[4] = {l[0], l[1], l[2], l[3]};
    if (__all(l[0] >= near && l[1] >= near && l[2] >= near && l[3] >= near)) {
      table_exp<false, 4>(x, m);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) m[e] = mass(l[e]);
    }
  }
};

// Inverse-CDF draw over the vocabulary: the first token, in token order, whose running sum of mass exceeds u times the
// total; -1 when the total is not positive.  for_blocks(f) calls f(block, t) for every block of this wave in ascending order
// (see wave_blocks); mass4(t, v) gives the masses of tokens v .. v+3 of that block (v = 256 block + 4 lane; 0 past the end)
// and must return the same values every time it is asked.  The masses are summed per segment, one wave finds the segment that holds the target,
// and the wave that owns it scans it.  Every thread of the workgroup calls it; the result is uniform.  All sums
// have a fixed order.
template <bool ONE, typename FB, typename F>  // ONE: a block per segment (rows of up to 262144 tokens)
__device__ __forceinline__ int cdf_draw(FB for_blocks, F mass4, int V, double u, DrawShared& sh, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  const int grp = ONE ? 1 : seg_blocks(V);
  const int n_blocks = (V + SV_BLOCK - 1) / SV_BLOCK, n_seg = (n_blocks + grp - 1) / grp;
  __syncthreads();  // (the shared arrays of an earlier draw have been read)
  if constexpr (ONE) {
    // the wave's eight segments are summed over the lanes together: every exchange with the lane 32, 16, 8 away halves the
    // segments a lane still carries (10 exchanges instead of 48)
    static_assert(SV_REG_TILES == 8, "three halvings");
    double s8[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for_blocks([&](int blk, int t) {
      double m[4];
      mass4(t, blk * SV_BLOCK + 4 * lane, m);
      s8[t] = (m[0] + m[1]) + (m[2] + m[3]);
    });
    double s4[4], s2[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) s4[i] = lane_halve_d<32>(s8[i], s8[4 + i]);
#pragma unroll
    for (int i = 0; i < 2; ++i) s2[i] = lane_halve_d<16>(s4[i], s4[2 + i]);
    const bool lo = lane & 8;
    double s = (lo ? s2[1] : s2[0]) + lane_swap_d<0x128>(lo ? s2[0] : s2[1]);  // row_ror:8
    s += lane_swap_d<LANE_1>(s);
    s += lane_swap_d<LANE_2>(s);
    s += lane_swap_d<LANE_4>(s);
    if ((lane & 7) == 0) sh.seg[(lane >> 3) * SV_WAVES + wave] = s;  // (segments past the row's end: zero)
  } else {
    double run = 0.0;
    for_blocks([&](int blk, int t) {
      double m[4];
      mass4(t, blk * SV_BLOCK + 4 * lane, m);
      run += (m[0] + m[1]) + (m[2] + m[3]);
      if (blk % grp == grp - 1 || blk == n_blocks - 1) {  // (wave-uniform)
        const double s = wave_sum_d(run);
        if (lane == 0) sh.seg[blk / grp] = s;
        run = 0.0;
      }
    });
  }
  __syncthreads();
  if (wave == 0) {
    const int per = (n_seg + 63) >> 6;
    double mine = 0.0;
    for (int i = 0; i < per; ++i) {
      const int s = lane * per + i;
      if (s < n_seg) mine += sh.seg[s];
    }
    const double inc = wave_scan_d(mine);
    const double total = lane_63_d(inc), target = u * total;
    double before = lane_before_d(inc);
    int hit = 0x7fffffff, last = -1;
    double hit_before = 0.0, last_before = 0.0;
    for (int i = 0; i < per; ++i) {
      const int s = lane * per + i;
      if (s >= n_seg) break;
      const double m = sh.seg[s];
      if (m > 0.0) {
        last = s;
        last_before = before;
        if (hit == 0x7fffffff && before + m > target) { hit = s; hit_before = before; }
      }
      before += m;
    }
    const unsigned long long any = __ballot(hit != 0x7fffffff), pos = __ballot(last >= 0);
    if (pos == 0ull) {                      // no mass anywhere (or not a number)
      if (lane == 0) sh.pick[0] = -1;
    } else if (any) {
      if (lane == __ffsll(any) - 1) { sh.pick[0] = hit; sh.target[0] = target - hit_before; }
    } else if (lane == 63 - __clzll(pos)) {  // rounding left the target at the end: the last segment with mass
      sh.pick[0] = last;
      sh.target[0] = target - last_before;
    }
    if (lane == 0) { sh.target[1] = total; sh.pick[1] = -1; }
  }
  __syncthreads();
  if (!(sh.target[1] > 0.0) || sh.pick[0] < 0) return -1;  // (whole workgroup)
  const int seg = sh.pick[0];
  if (wave == seg % SV_WAVES) {  // (the segment's own wave: it holds the masses)
    const double target = sh.target[0];
    double base = 0.0;
    int tok = -1, tail = -1;     // the token; the last token with mass so far
    for_blocks([&](int blk, int t) {
      if (blk / grp != seg || tok >= 0) return;
      const int v = blk * SV_BLOCK + 4 * lane;
      double m[4];
      mass4(t, v, m);
      const double mine = (m[0] + m[1]) + (m[2] + m[3]);
      const double inc = wave_scan_d(mine);
      const double sum = lane_63_d(inc);
      double cum = base + lane_before_d(inc);
      int hit = -1, last = -1;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        cum += m[e];
        if (m[e] > 0.0) {
          last = v + e;
          if (hit < 0 && cum > target) hit = v + e;
        }
      }
      const unsigned long long any = __ballot(hit >= 0), pos = __ballot(last >= 0);
      if (any) tok = __shfl(hit, __ffsll(any) - 1, 64);
      if (pos) tail = __shfl(last, 63 - __clzll(pos), 64);
      base += sum;
    });
    if (tok < 0) tok = tail;     // rounding left the target at the segment's end: its last token with mass
    if (lane == 0) sh.pick[1] = tok;
  }
  __syncthreads();
  return sh.pick[1];
}

// The blocks of this wave: block b of a row belongs to segment b / grp and so to wave (b / grp) % 16.
// TILES > 0: the row has at most TILES * 4096 tokens (grp == 1), the loop is unrolled and the block's index in the
// wave is a constant; TILES == 0: any row.
template <int TILES, typename F>
__device__ __forceinline__ void wave_blocks(int V, int wave, F f) {
  const int n_blocks = (V + SV_BLOCK - 1) / SV_BLOCK;
  if constexpr (TILES > 0) {
#pragma unroll
    for (int t = 0; t < TILES; ++t)
      if (t * SV_WAVES + wave < n_blocks) f(t * SV_WAVES + wave, t);
  } else {
    const int grp = seg_blocks(V);
    for (int s = wave; s * grp < n_blocks; s += SV_WAVES)
      for (int b = s * grp; b < min(n_blocks, (s + 1) * grp); ++b) f(b, 0);
  }
}

// Largest score of a row, then Z = sum_v exp((l_v - max) / T), both uniform over the workgroup; with TILES > 0 the
// exponentials stay in ex (zero past the end of the row).
template <int TILES>
__device__ __forceinline__ void row_max_and_z(const float* __restrict__ L, int V, Temp& temp, DrawShared& sh, int tid,
                                              double (&ex)[TILES > 0 ? TILES : 1][4], double& Z) {
  const int lane = tid & 63, wave = tid >> 6;
  double2 power = make_double2(0.0, 0.0);    // (asked for ahead of the row)
  if (tid < 64) power = make_double2(kPow2[2 * tid], kPow2[2 * tid + 1]);
  f32x4 raw[TILES > 0 ? TILES : 1];
  float mx = -INFINITY;
  wave_blocks<TILES>(V, wave, [&](int blk, int t) { raw[t] = load_row4(L, blk * SV_BLOCK + 4 * lane, V, -INFINITY);
                                                     if (TILES == 0) mx = fmaxf(mx, fmaxf(fmaxf(raw[0][0], raw[0][1]), fmaxf(raw[0][2], raw[0][3]))); });
  if constexpr (TILES > 0)
    wave_blocks<TILES>(V, wave, [&](int, int t) { mx = fmaxf(mx, fmaxf(fmaxf(raw[t][0], raw[t][1]), fmaxf(raw[t][2], raw[t][3]))); });
  mx = wave_max(mx);
  if (lane == 0) sh.redf[wave] = mx;
  if (tid < 64) sh.pow2[tid] = power;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < SV_WAVES; ++w) mx = fmaxf(mx, sh.redf[w]);
  temp.largest(mx);
  double zp = 0.0;
  wave_blocks<TILES>(V, wave, [&](int blk, int t) {
    const int v = blk * SV_BLOCK + 4 * lane;
    const f32x4 l = TILES > 0 ? raw[t] : load_row4(L, v, V, -INFINITY);
    temp.mass4(l, ex[t]);
    if ((blk + 1) * SV_BLOCK > V) {          // (wave-uniform)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (v + e >= V) ex[t][e] = 0.0;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) zp += ex[t][e];
  });
  zp = wave_sum_d(zp);
  if (lane == 0) sh.red[wave] = zp;
  __syncthreads();
  Z = 0.0;
#pragma unroll
  for (int w = 0; w < SV_WAVES; ++w) Z += sh.red[w];
}

// The top byte of the counter's last word names the consumer of the numbers, so that the verifier
// (0) and the drafting SSMs (1 + index) never share a stream under one seed; steps are below 2^56.
__device__ __forceinline__ void position_uniforms(uint32_t b, uint32_t j, uint32_t step_lo, uint32_t step_hi,
                                                  uint32_t consumer, uint32_t seed_lo, uint32_t seed_hi, double& u0,
                                                  double& u1) {
  uint32_t w[4] = {b, j, step_lo, (step_hi & 0x00ffffffu) | (consumer << 24)};
  philox4x32_10(w, seed_lo, seed_hi);
  u0 = unit_double(w[0], w[1]);
  u1 = unit_double(w[2], w[3]);
}

// One workgroup per (position j, sequence b).
template <int TILES>
__global__ void __launch_bounds__(SV_THREADS) verify_sample_kernel(
    const float* __restrict__ logits, const int32_t* __restrict__ voted, const float* __restrict__ draft_probs,
    const int32_t* __restrict__ spec_len, const int32_t* __restrict__ greedy, int B, int k_max, int M, int V,
    double temperature, double inv_temperature, uint32_t seed_lo, uint32_t seed_hi, uint32_t step_lo, uint32_t step_hi,
    int32_t* __restrict__ sampled, int32_t* dev_status) {
  __shared__ DrawShared sh;
  __shared__ int s_int[2];  // rows before this sequence, bad flag
  const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int32_t* out = sampled + (size_t)b * (k_max + 1) + j;

  if (tid < 2) s_int[tid] = 0;
  __syncthreads();
  {  // rows of the sequences before b (integer sum: order-free)
    int part = 0, bad = 0;
    for (int i = tid; i < b; i += SV_THREADS) {
      const int k = spec_len[i];
      if (k < 0 || k > k_max) bad = 1;
      part += k + 1;
    }
    if (part) atomicAdd(&s_int[0], part);
    if (bad) atomicOr(&s_int[1], 1);
  }
  __syncthreads();
  const int k_b = spec_len[b];
  const int row = s_int[0] + j;
  const bool seq_ok = !s_int[1] && k_b >= 0 && k_b <= k_max && greedy[(size_t)b * (k_max + 1)] >= 0;
  if (!seq_ok || j > k_b || row >= M) {  // (whole workgroup)
    if (tid == 0) {
      *out = -1;
      if (seq_ok && j <= k_b && dev_status) atomicOr(dev_status, MN_DEV_SPEC_LEN);  // rows do not add up to M
    }
    return;
  }
  const float* L = logits + (size_t)row * V;
  Temp temp{temperature, inv_temperature, inv_temperature * 0x1.71547652b82fep+6, sh.pow2, 0.0, -800.0 * temperature, 1.0 / 120.0, 0.f};  // 64 / ln2
  double ex[TILES > 0 ? TILES : 1][4];
  double Z;
  row_max_and_z<TILES>(L, V, temp, sh, tid, ex, Z);
  double u_acc, u_res;
  position_uniforms((uint32_t)b, (uint32_t)j, step_lo, step_hi, 0u, seed_lo, seed_hi, u_acc, u_res);

  // ---- does the speculated token survive? ----
  bool keep = false;
  int x = -1;
  const float* Q = nullptr;
  if (j < k_b) {
    x = voted[(size_t)b * k_max + j];
    Q = draft_probs + ((size_t)b * k_max + j) * V;
    if (x >= 0 && x < V) {
      const double ox = temp.mass(L[x]) / Z;
      const double qx = (double)Q[x];
      keep = (qx <= ox) || (u_acc < ox / qx);
    }
  }
  if (keep) {  // (whole workgroup: x, Q, Z, the random numbers are uniform over it)
    if (tid == 0) *out = x;
    return;
  }
  // ---- a token from max(0, o - q); without q (position k_b) from o.  When nothing of o lies above q (a q that
  // sums above 1) the replacement comes from o without the rejected token, so that it still differs from what
  // it replaces (the acceptance reads "first entry that differs" as the first rejection); and when all of o
  // sits on that token there is nothing else to emit: it stays ----
  const double inv_z = 1.0 / Z;  // (Z >= 1: the largest score contributes exp(0))
  auto o4 = [&](int v, double (&o)[4]) {  // probabilities of tokens v .. v+3, recomputed from the scores
    const f32x4 l = load_row4(L, v, V, -INFINITY);
    temp.mass4(l, o);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = v + e < V ? div_by(o[e], Z, inv_z) : 0.0;
  };
  int tok = -1;
  if constexpr (TILES > 0) {
    // the masses take the place of the exponentials in the registers
    wave_blocks<TILES>(V, wave, [&](int blk, int t) {
      f32x4 q = {0.f, 0.f, 0.f, 0.f};
      if (Q) q = load_row4(Q, blk * SV_BLOCK + 4 * lane, V, 0.f);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double o = div_by(ex[t][e], Z, inv_z);
        ex[t][e] = Q ? fmax(0.0, o - (double)q[e]) : o;
      }
    });
    tok = cdf_draw<(TILES > 0)>([&](auto f) { wave_blocks<TILES>(V, wave, f); },
                   [&](int t, int, double (&m)[4]) { m[0] = ex[t][0]; m[1] = ex[t][1]; m[2] = ex[t][2]; m[3] = ex[t][3]; },
                   V, u_res, sh, tid);
  } else {
    tok = cdf_draw<false>([&](auto f) { wave_blocks<0>(V, wave, f); },
                   [&](int, int v, double (&m)[4]) {
                     o4(v, m);
                     if (Q) {
                       const f32x4 q = load_row4(Q, v, V, 0.f);
#pragma unroll
                       for (int e = 0; e < 4; ++e) m[e] = fmax(0.0, m[e] - (double)q[e]);
                     }
                   },
                   V, u_res, sh, tid);
  }
  if (Q && tok < 0) {
    tok = cdf_draw<false>([&](auto f) { wave_blocks<0>(V, wave, f); },
                   [&](int, int v, double (&m)[4]) {
                     o4(v, m);
#pragma unroll
                     for (int e = 0; e < 4; ++e)
                       if (v + e == x) m[e] = 0.0;
                   },
                   V, u_res, sh, tid);
    if (tok < 0) tok = x;
  }
  if (tid == 0) *out = tok;
}

// One workgroup per sequence: token ~ q = softmax(scores / T) of a drafting SSM, and q itself in fp32.
// The draw is taken from the fp32 values that are written out, so what the verifier is later told is
// exactly the distribution the token came from.
template <int TILES>
__global__ void __launch_bounds__(SV_THREADS) draft_sample_kernel(const float* __restrict__ logits, int V,
                                                                  double temperature, double inv_temperature,
                                                                  uint32_t seed_lo, uint32_t seed_hi,
                                                                  uint32_t step_lo, uint32_t step_hi, uint32_t consumer,
                                                                  uint32_t t_pos, int32_t* __restrict__ tokens,
                                                                  long token_stride, float* __restrict__ probs,
                                                                  long probs_stride) {
  __shared__ DrawShared sh;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float* L = logits + (size_t)b * V;
  Temp temp{temperature, inv_temperature, inv_temperature * 0x1.71547652b82fep+6, sh.pow2, 0.0, -800.0 * temperature, 1.0 / 120.0, 0.f};  // 64 / ln2
  double ex[TILES > 0 ? TILES : 1][4];
  double Z;
  row_max_and_z<TILES>(L, V, temp, sh, tid, ex, Z);
  double u_unused, u;
  position_uniforms((uint32_t)b, t_pos, step_lo, step_hi, consumer, seed_lo, seed_hi, u_unused, u);
  const double inv_z = 1.0 / Z;
  auto q4 = [&](int v, double (&m)[4]) {  // the fp32 probabilities of tokens v .. v+3
    const f32x4 l = load_row4(L, v, V, -INFINITY);
    temp.mass4(l, m);
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = v + e < V ? (double)(float)div_by(m[e], Z, inv_z) : 0.0;
  };
  float* P = probs ? probs + (size_t)b * probs_stride : nullptr;
  wave_blocks<TILES>(V, wave, [&](int blk, int t) {
    const int v = blk * SV_BLOCK + 4 * lane;
    double m[4];
    if constexpr (TILES > 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) m[e] = ex[t][e] = (double)(float)div_by(ex[t][e], Z, inv_z);
    } else if (P) {
      q4(v, m);
    }
    if (P) {
      if (v + 3 < V) {
        *reinterpret_cast<f32x4_u*>(P + v) = (f32x4_u){(float)m[0], (float)m[1], (float)m[2], (float)m[3]};
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (v + e < V) P[v + e] = (float)m[e];
      }
    }
  });
  int tok;
  if constexpr (TILES > 0)
    tok = cdf_draw<(TILES > 0)>([&](auto f) { wave_blocks<TILES>(V, wave, f); },
                   [&](int t, int, double (&m)[4]) { m[0] = ex[t][0]; m[1] = ex[t][1]; m[2] = ex[t][2]; m[3] = ex[t][3]; },
                   V, u, sh, tid);
  else
    tok = cdf_draw<false>([&](auto f) { wave_blocks<0>(V, wave, f); },
                   [&](int, int v, double (&m)[4]) {
                     if (P && v + 3 < V) {  // (this thread wrote them itself: cheaper than the exponentials again)
                       const f32x4_u q = *reinterpret_cast<const f32x4_u*>(P + v);
                       m[0] = (double)q[0]; m[1] = (double)q[1]; m[2] = (double)q[2]; m[3] = (double)q[3];
                     } else {
                       q4(v, m);
                     }
                   },
                   V, u, sh, tid);
  if (tid == 0) tokens[(size_t)b * token_stride] = tok;
}

// 1 / T where both are comfortably normal numbers, 0 otherwise (the kernels then divide)
static double temperature_reciprocal(double T) { return T > 0x1p-100 && T < 0x1p100 ? 1.0 / T : 0.0; }

void launch_verify_sample(const float* logits, const int32_t* voted, const float* draft_probs, const int32_t* spec_len,
                          const int32_t* greedy, int B, int k_max, int M, int V, double temperature, uint64_t seed,
                          uint64_t step, int32_t* sampled, int32_t* dev_status, hipStream_t st) {
  if (B <= 0) return;
  auto* kernel = V <= SV_REG_TILES * SV_TILE ? verify_sample_kernel<SV_REG_TILES> : verify_sample_kernel<0>;
  kernel<<<dim3(k_max + 1, B), SV_THREADS, 0, st>>>(
      logits, voted, draft_probs, spec_len, greedy, B, k_max, M, V, temperature, temperature_reciprocal(temperature),
      (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32), sampled, dev_status);
}

void launch_draft_sample(const float* logits, int B, int V, double temperature, uint64_t seed, uint64_t step, int ssm,
                         int t_pos, int32_t* tokens, long token_stride, float* probs, long probs_stride, hipStream_t st) {
  if (B <= 0) return;
  auto* kernel = V <= SV_REG_TILES * SV_TILE ? draft_sample_kernel<SV_REG_TILES> : draft_sample_kernel<0>;
  kernel<<<B, SV_THREADS, 0, st>>>(logits, V, temperature, temperature_reciprocal(temperature), (uint32_t)seed,
                                   (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32), (uint32_t)(1 + ssm),
                                   (uint32_t)t_pos, tokens, token_stride, probs, probs_stride);
}

int verify_sample_max_vocab() { return SV_MAX_VOCAB; }

}  // namespace mn
