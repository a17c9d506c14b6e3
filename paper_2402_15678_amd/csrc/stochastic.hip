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

#include <cmath>

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
// exponentials of one row on one CU (15 vector instructions of four cycles per token and lane: 3.1 us for 32000 tokens) and by
// the chain load -> exponentials -> sum -> masses -> draw, so a row is read once, every exponential is computed once, and the workgroup
// meets twice: for the sum of the exponentials and for the sums of the segments.  Measured at 32000 tokens: 13.2 us for the 144 positions of 16
// requests and 11.8 us for 16 drafted tokens (18.3 and 13.7 with the exponentials relative to the row's largest score, a third meeting of the workgroup, and the
// masses divided by Z).
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
__device__ __forceinline__ int wave_of(int tid) { return __builtin_amdgcn_readfirstlane(tid >> 6); }  // (scalar: its branches and addresses are)
__device__ __forceinline__ int seg_blocks(int V) { return (V + SV_MAX_SEGS * SV_BLOCK - 1) / (SV_MAX_SEGS * SV_BLOCK); }

// (rows start at any multiple of 4 bytes: the vocabulary need not be a multiple of 4)
// this lane's four consecutive values of block blk (uniform) of a row, `pad` past its end
__device__ __forceinline__ f32x4 load_row4(const float* __restrict__ R, int blk, int lane, int V, float pad) {
  const int v = blk * SV_BLOCK + 4 * lane;
  if ((blk + 1) * SV_BLOCK <= V || v + 3 < V) {
    const f32x4_u x = *reinterpret_cast<const f32x4_u*>(R + (size_t)blk * SV_BLOCK + 4 * lane);
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
  double2 pow2[256];          // (see PowerLoad)
  double red[SV_WAVES];
  int ref[SV_WAVES];
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

// 2^(j/256), j = 0 .. 3
__device__ const double kPow2Fine[8] = {0x1.0000000000000p+0, 0x0.0p+0, 0x1.00b1afa5abcbfp+0, -0x1.4f6b2a7609f71p-55,
                                        0x1.0163da9fb3335p+0, 0x1.b61299ab8cdb7p-54, 0x1.02168143b0281p+0, -0x1.2bf310fc54eb6p-55};

// The table in LDS: for every j = 0 .. 255 a double c next to 2^(j/256) and what it leaves over, 2^(j/256) / c - 1.  The high word of c
// has j << 12 taken off (Temp adds the power of two and the index back in one step).
struct PowerLoad {
  double2 a, b;
  __device__ __forceinline__ void ask(int tid) {
    const int j = tid & 255;
    a = make_double2(kPow2[2 * (j >> 2)], kPow2[2 * (j >> 2) + 1]);
    b = make_double2(kPow2Fine[2 * (j & 3)], kPow2Fine[2 * (j & 3) + 1]);
  }
  __device__ __forceinline__ void store(DrawShared& sh, int tid) const {
    if (tid >= 256) return;
    const double c = a.x * b.x, left = fma(a.x, b.x, -c) + (a.x * b.y + a.y * b.x);
    sh.pow2[tid] = make_double2(__hiloint2double(__double2hiint(c) - (tid << 12), __double2loint(c)), (double)((float)left / (float)c));
  }
};

// A place that the values pass in program order: without it the compiler takes one operation of every token of the row after the other,
// and the intermediate values of all of them do not fit the registers (280 spilled; 60000 cycles for the row's exponentials instead of 8000).  As one
// value: apart, they stay where the reads of the table put one half of each, and in between no piece of a row fits (22 spilled).
template <typename T>
__device__ __forceinline__ void in_turn(T& a, T& b, T& c, T& d) {
  T __attribute__((ext_vector_type(4))) v = {a, b, c, d};
  asm volatile("" : "+v"(v));
  a = v[0]; b = v[1]; c = v[2]; d = v[3];
}

// the next float at or above x
__device__ __forceinline__ float float_above(double x) {
  const float n = (float)x;
  if (!((double)n < x)) return n;
  return n == 0.f ? 1e-45f : __uint_as_float(__float_as_uint(n) + (n > 0.f ? 1 : -1));
}
constexpr double ROUND_MAGIC = 6755399441055744.0;  // 1.5 * 2^52: added to a number, its nearest whole number sits in the low bits

// Exponentials of scores at temperature T, table-driven (P. T. P. Tang, ACM TOMS 15(2), 1989): l / T = (n + f) ln2/256 with n whole
// and |f| <= 1/2, and exp(l / T) = 2^(n >> 8) * 2^((n & 255)/256) * (1 + a1 f + .. + a4 f^4), the fifth-order term spread over a1 and a3.
// f comes out of two fmas with k = 256 / (T ln2) in two pieces, so nothing is lost to the reciprocal of T.  (Several copies of the table, so
// that the lanes of a read spread over the banks, change nothing: 8040 cycles for a row of 32768 tokens with one copy and with eight, 5940 without the table.)
// Relative error against 128-bit arithmetic, 200000 arguments in [-20, 0] at each of five temperatures: rms 4.7e-17, largest 1.1e-16, what a correctly
// rounded exponential has (4.8e-17 and 1.4e-16 at T = 1, 5e-16 and 1e-15 elsewhere with a reciprocal of T in one piece).
// About half the instructions of the general function, which is most of these kernels' time.
// A wave takes the exponentials relative to a power of two of its own, at or above its largest one (`relative_to`): nobody waits for
// the largest score of the row, and the waves' sums are brought to one scale exactly.  Where that does not work - scores that are not numbers or,
// from SV_LOW_T on, of a size that leaves n no room, rows beyond SV_MAX_FAR - they are taken relative to the row's largest score (`below`),
// and for temperatures so extreme that the reciprocal leaves the normal range (inv == 0) by the general function and a
// division.  Scores more than 800 T below the largest are cut there (the exponential is zero long before), so that a masked token (minus
// infinity) stays finite; NaN passes through.  The cut is on fp64 numbers: 800 T may be far below the spacing of the scores in fp32,
// and the largest score may be the type's lowest value.
struct Temp {
  double T, inv, k, k_lo;
  const double2* table;
  double a4;                 // (in vector registers, as k: an instruction reads one scalar constant)
  double base;               // taken off the scores (below)
  double magic;              // ROUND_MAGIC less the reference (relative_to)
  double lowest;             // of a score, less base
  float near = INFINITY;     // scores from here on are within 690 T of the largest (see mass4); NaN or more than any score: none are

  __device__ __forceinline__ Temp(double t, double inv_t, double kh, double kl, const DrawShared& sh)
      : T(t), inv(inv_t), k(kh), k_lo(kl), table(sh.pow2), a4(0x1.3b2ab6fba4e77p-39) {
    asm("" : "+v"(k), "+v"(a4));
  }
  __device__ __forceinline__ void below(float mx) {  // mx the row's largest score
    base = (double)mx;
    magic = ROUND_MAGIC;
    lowest = -800.0 * T;
    near = inv == 0.0 ? INFINITY : float_above(base - 690.0 * T);
  }
  __device__ __forceinline__ void relative_to(int e, double mx) {  // 2^e, mx the largest score (or more)
    base = 0.0;
    magic = ROUND_MAGIC - 256.0 * (double)e;
    magic = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(magic)), __builtin_amdgcn_readfirstlane(__double2loint(magic)));
    lowest = mx - 800.0 * T;
    near = float_above(mx - 690.0 * T);
  }
  // N exponentials side by side (one is a chain of eleven dependent operations and an LDS read).  SMALL: a result may be below the
  // normal range, an argument below the cut or not a number.
  template <bool SMALL, int N>
  __device__ __forceinline__ void powers(double (&x)[N], double (&m)[N]) const {
    double t[N], nd[N], f[N], p[N];
    double2 c[N];
    int n[N];
    if (SMALL) {
#pragma unroll
      for (int e = 0; e < N; ++e) x[e] = x[e] < lowest ? lowest : x[e];
    }
#pragma unroll
    for (int e = 0; e < N; ++e) t[e] = fma_vvs(x[e], k, magic);
#pragma unroll
    for (int e = 0; e < N; ++e) n[e] = (int)(uint32_t)__double_as_longlong(t[e]);
#pragma unroll
    for (int e = 0; e < N; ++e) c[e] = table[n[e] & 255];
#pragma unroll
    for (int e = 0; e < N; ++e) nd[e] = t[e] - magic;
#pragma unroll
    for (int e = 0; e < N; ++e) f[e] = fma(x[e], k, -nd[e]);
#pragma unroll
    for (int e = 0; e < N; ++e) f[e] = fma(x[e], k_lo, f[e]);
#pragma unroll
    for (int e = 0; e < N; ++e) p[e] = fma_vvs(f[e], a4, 0x1.c6b090da1e082p-29);  // (ln2/256)^i / i!, the fifth one folded into the third and first
#pragma unroll
    for (int e = 0; e < N; ++e) p[e] = fma_vvs(f[e], p[e], 0x1.ebfbdff82c58fp-19);
#pragma unroll
    for (int e = 0; e < N; ++e) p[e] = fma_vvs(f[e], p[e], 0x1.62e42fefa39b9p-9);
#pragma unroll
    for (int e = 0; e < N; ++e) p[e] = fma(f[e], p[e], c[e].y);
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const double s = __hiloint2double(__double2hiint(c[e].x) + ((SMALL ? n[e] & 255 : n[e]) << 12), __double2loint(c[e].x));
      const double y = fma(s, p[e], s);
      m[e] = SMALL ? ldexp(y, n[e] >> 8) : y;
    }
  }
  template <bool BELOW>
  __device__ __forceinline__ double mass(float l) const {
    if (BELOW && inv == 0.0) return exp(((double)l - base) / T);  // (uniform)
    double x[1] = {BELOW ? (double)l - base : (double)l}, m[1];
    powers<true, 1>(x, m);
    return m[0];
  }
  // The masses of four scores, bit for bit those of mass().  PLAIN: every one of them is within 690 T of the largest (>= near): the
  // powers of two are added to the exponent field and nothing is cut.
  template <bool BELOW, bool PLAIN>
  __device__ __forceinline__ void mass4(const f32x4& l, double (&m)[4]) const {
    if (BELOW && inv == 0.0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) m[e] = mass<BELOW>(l[e]);
      return;
    }
#pragma unroll
    for (int e = 0; e < 4; e += 2) {
      if (e) asm volatile("" : "+v"(m[0]), "+v"(m[1]));
      double x[2] = {BELOW ? (double)l[e] - base : (double)l[e], BELOW ? (double)l[e + 1] - base : (double)l[e + 1]}, y[2];
      powers<!PLAIN, 2>(x, y);
      m[e] = y[0];
      m[e + 1] = y[1];
    }
  }
  template <bool BELOW>
  __device__ __forceinline__ void mass4(const f32x4& l, double (&m)[4]) const {
    if (__all(l[0] >= near && l[1] >= near && l[2] >= near && l[3] >= near)) mass4<BELOW, true>(l, m);
    else mass4<BELOW, false>(l, m);
  }
};

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

// The segment that holds u times the total mass, with the target inside it, found by one wave from the segments' masses (per
// of them in a lane, in order; those above `floor` count as mass); false when there is no mass (or it is not a number).
struct Hit {
  int seg;
  double target, total;
};
__device__ __forceinline__ double lane_any_d(double v, int lane) {  // (lane uniform)
  return both_halves(v, [&](uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)x, lane); });
}
__device__ __forceinline__ bool find_segment(const double* seg, int n_seg, int per, double u, double floor, int lane, Hit& h) {
  double mine = 0.0;
  for (int i = 0; i < per; ++i) {
    const int s = lane * per + i;
    if (s < n_seg) mine += seg[s];
  }
  const double inc = wave_scan_d(mine);
  const double total = lane_63_d(inc), target = u * total;
  double before = lane_before_d(inc);
  int hit = -1, last = -1;
  double hit_before = 0.0, last_before = 0.0;
  for (int i = 0; i < per; ++i) {
    const int s = lane * per + i;
    const double m = s < n_seg ? seg[s] : 0.0;
    if (m > floor) {
      last = s;
      last_before = before;
      if (hit < 0 && before + m > target) { hit = s; hit_before = before; }
    }
    before += m;
  }
  const unsigned long long any = __ballot(hit >= 0), pos = __ballot(last >= 0);
  h.total = total;
  h.seg = -1;
  h.target = 0.0;
  if (pos == 0ull) return false;
  const int from = any ? __ffsll(any) - 1 : 63 - __clzll(pos);  // (rounding may leave the target at the end: the last segment with mass)
  h.seg = __builtin_amdgcn_readlane(any ? hit : last, from);
  h.target = target - lane_any_d(any ? hit_before : last_before, from);
  return true;
}
// One block of the segment: sets tok to the token that the running sum (base before the block) passes the target in, tail to the
// last token with mass; returns the block's mass.
__device__ __forceinline__ double find_token(const double (&m)[4], int v, double base, double target, double floor, int& tok, int& tail) {
  const double inc = wave_scan_d((m[0] + m[1]) + (m[2] + m[3]));
  double cum = base + lane_before_d(inc);
  int hit = -1, last = -1;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    cum += m[e];
    if (m[e] > floor) {
      last = v + e;
      if (hit < 0 && cum > target) hit = v + e;
    }
  }
  const unsigned long long any = __ballot(hit >= 0), pos = __ballot(last >= 0);
  if (any) tok = __builtin_amdgcn_readlane(hit, __ffsll(any) - 1);
  if (pos) tail = __builtin_amdgcn_readlane(last, 63 - __clzll(pos));
  return lane_63_d(inc);
}

// RowRegs: nothing below it counts; a row with nothing above it is drawn from in the general form.  It is above all that the registers' form gives a
// wrong mass: scores cut at 690 T below their wave's largest (the cut is a float, and the spacing of the scores may be 88 T, so that they stand at 601 T,
// 2^-867) and waves left out beside the row's largest (2^-687 in all: 850 powers of two below it, a score behind the registers up to 145 above its
// wave's reference, 2^18 of them).
constexpr double MASS_FLOOR = 0x1p-600;
// RowRegs: a wave whose scores are all masked, with minus infinity or with a number so low (|score / T| 256 / ln2 >= 2^38) that nothing of it is left beside
// a row's power of two from ROW_LOW on; a row that is not for it
constexpr int ROW_NONE = -(1 << 30), ROW_LOW = ROW_NONE + 1024, ROW_GENERAL = 1 << 30;

// Inverse-CDF draw over the vocabulary: the first token, in token order, whose running sum of mass exceeds u times the
// total; -1 when the total is not positive.  mass4(blk, m) gives the masses of this lane's four tokens of block blk (0 past the end)
// and must return the same values every time it is asked.  The masses are summed per segment, one wave finds the segment that holds the target,
// and the wave that owns it scans it.  Every thread of the workgroup calls it; the result is uniform.  All sums
// have a fixed order.
template <typename F>
__device__ __forceinline__ int cdf_draw(F mass4, int V, double u, DrawShared& sh, int tid) {
  const int lane = tid & 63, wave = wave_of(tid);
  const int grp = seg_blocks(V);
  const int n_blocks = (V + SV_BLOCK - 1) / SV_BLOCK, n_seg = (n_blocks + grp - 1) / grp;
  __syncthreads();  // (the shared arrays of an earlier draw have been read)
  double run = 0.0;
  wave_blocks<0>(V, wave, [&](int blk, int) {
    double m[4];
    mass4(blk, m);
    run += (m[0] + m[1]) + (m[2] + m[3]);
    if (blk % grp == grp - 1 || blk == n_blocks - 1) {  // (wave-uniform)
      const double s = wave_sum_d(run);
      if (lane == 0) sh.seg[blk / grp] = s;
      run = 0.0;
    }
  });
  __syncthreads();
  if (wave == 0) {
    Hit h;
    const bool any = find_segment(sh.seg, n_seg, (n_seg + 63) >> 6, u, 0.0, lane, h);
    if (lane == 0) {
      sh.pick[0] = any ? h.seg : -1;
      sh.pick[1] = -1;
      sh.target[0] = h.target;
      sh.target[1] = h.total;
    }
  }
  __syncthreads();
  if (!(sh.target[1] > 0.0) || sh.pick[0] < 0) return -1;  // (whole workgroup)
  const int seg = sh.pick[0];
  if (wave == seg % SV_WAVES) {  // (the segment's own wave)
    const double target = sh.target[0];
    double base = 0.0;
    int tok = -1, tail = -1;     // the token; the last token with mass so far
    wave_blocks<0>(V, wave, [&](int blk, int) {
      if (blk / grp != seg || tok >= 0) return;
      double m[4];
      mass4(blk, m);
      base += find_token(m, blk * SV_BLOCK + 4 * lane, base, target, 0.0, tok, tail);
    });
    if (tok < 0) tok = tail;     // rounding left the target at the segment's end: its last token with mass
    if (lane == 0) sh.pick[1] = tok;
  }
  __syncthreads();
  return sh.pick[1];
}

// The exponentials of a row of up to TILES * 4096 tokens, in registers.  MORE: those of the tiles behind them are computed when they are asked for
// (`far`): once for their sum, once for their masses, and for the block that holds the draw.  SHIFT: scores are taken less the row's largest, in fp32, which
// is exact down to half of it (or twice, below zero); what lies beyond is far below any cut at the temperatures that this is for (see MN_ROW_KERNEL).
template <int TILES, bool MORE, bool SHIFT>
struct RowRegs {
  double ex[TILES][4];        // relative to this wave's power of two; zero past the end of the row (anything finite in a wave that is dead)
  int e_all;                  // the row's power of two: the largest of the waves'
  int down;                   // this wave's, less the row's: at most 0
  bool dead;                  // nothing of this wave is left beside the row's largest
  float shift = 0.f;          // taken off every score
  double Z, z_wave;           // sum of the row's exponentials relative to the row's power of two and to this wave's

  // the row may end in tile t (SHIFT: rows of fewer tiles take this form too)
  static constexpr __device__ bool may_end(int t) { return !MORE && (SHIFT || t == TILES - 1); }
  // A block's values of this lane, asked for whatever the row's length (V >= 4): blocks past the last repeat it, pieces that reach past the
  // end hold the last four values and are put in place afterwards (where V is no multiple of 4; what lies past the end is another value of the row).
  static __device__ __forceinline__ int first_of(int t, int wave, int lane, int V) {
    return min(t * SV_WAVES + wave, (V + SV_BLOCK - 1) / SV_BLOCK - 1) * SV_BLOCK + 4 * lane;
  }
  static __device__ __forceinline__ f32x4 ask(const float* __restrict__ R, int t, int wave, int lane, int V) {
    const f32x4_u x = *reinterpret_cast<const f32x4_u*>(R + min(first_of(t, wave, lane, V), V - 4));
    return (f32x4){x[0], x[1], x[2], x[3]};
  }
  static __device__ __forceinline__ f32x4 in_place(const f32x4& x, int t, int wave, int lane, int V) {
    const int past = first_of(t, wave, lane, V) - (V - 4);
    return (f32x4){past == 1 ? x[1] : past == 2 ? x[2] : past == 3 ? x[3] : x[0], past == 1 ? x[2] : past == 2 ? x[3] : x[1],
                   past == 1 ? x[3] : x[2], x[3]};
  }
  // masses of four scores of tile t, relative to the wave's power of two
  static __device__ __forceinline__ void masses(f32x4 l, int t, int wave, int lane, int V, const Temp& temp, double (&m)[4]) {
    const int blk = t * SV_WAVES + wave;
#pragma unroll
    for (int i = 0; i < 4; ++i) l[i] = fmaxf(l[i], temp.near);
    temp.template mass4<false, true>(l, m);
    if ((blk + 1) * SV_BLOCK > V) {            // (wave-uniform)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (blk * SV_BLOCK + 4 * lane + i >= V) m[i] = 0.0;
    }
  }
  __device__ __forceinline__ void shifted(f32x4& l) const {
    if constexpr (SHIFT) {
#pragma unroll
      for (int i = 0; i < 4; ++i) l[i] -= shift;
    }
  }
  __device__ __forceinline__ void far(const float* __restrict__ L, int t, int wave, int lane, int V, const Temp& temp, double (&m)[4]) const {
    f32x4 l = in_place(ask(L, t, wave, lane, V), t, wave, lane, V);
    shifted(l);
    masses(l, t, wave, lane, V, temp, m);
  }
  __device__ __forceinline__ void clear_past_end(int t, int wave, int lane, int V) {
    const int blk = t * SV_WAVES + wave;
    if ((blk + 1) * SV_BLOCK > V) {            // (wave-uniform)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (blk * SV_BLOCK + 4 * lane + i >= V) ex[t][i] = 0.0;
    }
  }

  // The power of two that a wave takes its exponentials relative to, the next one at or above its largest (mx: each lane's largest score, which becomes the
  // wave's; a NaN stays)
  static __device__ __forceinline__ int reference(float& mx, Temp& temp) {
    const bool nan = __any(mx != mx);
    mx = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(wave_max(mx))));
    const double top = (double)mx * temp.k;
    const bool ok = __all(__builtin_fabs(top) < 0x1p38) && !nan;
    const int e = ok ? __builtin_amdgcn_readfirstlane((int)ceil(top * (1.0 / 256.0))) : mx > 0.f || nan ? ROW_GENERAL : ROW_NONE;
    temp.relative_to(ok ? e : 0, ok ? (double)mx : 0.0);
    return e;
  }
  // Scores up to here may be taken relative to a wave's power of two: a float at or below 100 T above the largest that it was chosen for (rounded to the nearest
  // it could be 133 T)
  static __device__ __forceinline__ float room_above(float mx, int e, const Temp& temp) {
    return e == ROW_NONE ? mx : -float_above(-((double)mx + 100.0 * temp.T));
  }

  // Uniform result; false: the row has scores that are not numbers, or too large for this (or none that is not masked).
  // Scores more than 690 T below the wave's largest count as that far below: MASS_FLOOR and the draw tell them from mass.
  // soon: another row (or null) that the kernel may read next; a line of it per thread is on its way to the L2 while the exponentials are
  // computed.  (Asked for beside the scores it holds them up: 1 us of 16 at 144 rows.)
  __device__ __forceinline__ bool load(const float* __restrict__ L, const float* __restrict__ soon, int V, Temp& temp, const PowerLoad& power, DrawShared& sh, int tid) {
    const int lane = tid & 63, wave = wave_of(tid), n_blocks = (V + SV_BLOCK - 1) / SV_BLOCK;
    f32x4 raw[TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) raw[t] = ask(L, t, wave, lane, V);
    power.store(sh, tid);
    if (!SHIFT) __syncthreads();
    if (V & 3) {
#pragma unroll
      for (int t = 0; t < TILES; ++t)
        if (may_end(t)) raw[t] = in_place(raw[t], t, wave, lane, V);
    }
    float mx = raw[0][0];                      // (a NaN stays)
#pragma unroll
    for (int i = 1; i < 4 * TILES; ++i) mx = __builtin_elementwise_maximum(mx, raw[i / 4][i % 4]);
    if constexpr (SHIFT) {
      float top = mx;
      if constexpr (MORE) {
        for (int t = TILES; t * SV_WAVES < n_blocks; ++t) {
          const f32x4 l = ask(L, t, wave, lane, V);
          top = fmaxf(top, fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3])));
        }
      }
      top = wave_max(top);
      if (lane == 0) sh.redf[wave] = top;
      __syncthreads();
      shift = sh.redf[0];
#pragma unroll
      for (int w = 1; w < SV_WAVES; ++w) shift = fmaxf(shift, sh.redf[w]);
      shift = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(shift)));  // (one that is not finite makes scores that are not numbers)
      mx -= shift;
    }
    int e = reference(mx, temp);
    float touch = 0.f;
    if (soon && 32 * tid < V) touch = soon[32 * tid];
    if (MORE && soon && 32 * (SV_THREADS + tid) < V) touch += soon[32 * (SV_THREADS + tid)];
    double zp = 0.0;
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      asm volatile("" : "+v"(raw[t]));         // (see in_turn)
      shifted(raw[t]);
      masses(raw[t], t, wave, lane, V, temp, ex[t]);
      in_turn(ex[t][0], ex[t][1], ex[t][2], ex[t][3]);
      zp += (ex[t][0] + ex[t][1]) + (ex[t][2] + ex[t][3]);
    }
    if constexpr (MORE) {
      // The tiles behind the registers keep the reference up to 100 T above the scores it was taken from: exponentials up to 2^145 leave room for z_wave.  A tile with
      // more moves it, and what has been computed with it.
      float above = room_above(mx, e, temp);
      f32x4 next = ask(L, TILES, wave, lane, V);
      for (int t = TILES; t * SV_WAVES + wave < n_blocks; ++t) {
        f32x4 l = in_place(next, t, wave, lane, V);
        shifted(l);
        next = ask(L, t + 1, wave, lane, V);
        float hi = __builtin_elementwise_maximum(__builtin_elementwise_maximum(l[0], l[1]), __builtin_elementwise_maximum(l[2], l[3]));
        if (__any(!(hi <= above)) && e != ROW_GENERAL) {
          const int was = e;
          e = reference(hi, temp);
          above = room_above(hi, e, temp);
          const double scale = was == ROW_NONE ? 0.0 : ldexp(1.0, was - e);
          zp *= scale;
#pragma unroll
          for (int i = 0; i < 4 * TILES; ++i) ex[i / 4][i % 4] *= scale;
        }
        double m[4];
        masses(l, t, wave, lane, V, temp, m);
        zp += (m[0] + m[1]) + (m[2] + m[3]);
      }
    }
    asm volatile("" ::"v"(touch));
    zp = wave_sum_d(zp);
    if (e == ROW_NONE) zp = 0.0;               // (wave-uniform; what ex holds then is not used)
    if (lane == 0) {
      sh.red[wave] = zp;
      sh.ref[wave] = e;
    }
    __syncthreads();
    e_all = sh.ref[0];
#pragma unroll
    for (int w = 1; w < SV_WAVES; ++w) e_all = max(e_all, sh.ref[w]);
    if (e_all == ROW_GENERAL || e_all < ROW_LOW) return false;
    Z = 0.0;
#pragma unroll
    for (int w = 0; w < SV_WAVES; ++w) Z += ldexp(sh.red[w], sh.ref[w] - e_all);
    if (!(Z > 0.0 && Z < INFINITY)) return false;
    down = e - e_all;
    z_wave = ldexp(Z, -down);
    dead = down < -850;
    if (dead) {                                // (ex stays: the verifier's sums of segments become zero by `down`, the drafter multiplies by zero)
      down = -4096;
      z_wave = 1.0;
    }
    return true;
  }

  // Inverse-CDF draw as cdf_draw, over the masses ex * 2^down: false when there is no mass, otherwise the wave that owns the token gets it (>= 0) in tok.
  // Every wave finds the segment for itself: the sums it needs are the only thing that the workgroup waits for.
  // more(t, first, m): the masses of a tile behind the registers; first: asked for the first time.
  template <typename F>
  __device__ __forceinline__ bool draw(int V, double u, int down_by, DrawShared& sh, int tid, int& tok, F more) {
    // the wave's eight segments are summed over the lanes together: every exchange with the lane 32, 16, 8 away halves the
    // segments a lane still carries (10 exchanges instead of 48)
    static_assert(TILES <= 8, "three halvings");
    const int lane = tid & 63, wave = wave_of(tid);
    const int n_blocks = (V + SV_BLOCK - 1) / SV_BLOCK;
    double s8[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < TILES; ++t) s8[t] = (ex[t][0] + ex[t][1]) + (ex[t][2] + ex[t][3]);
    auto store = [&](int t0, int tiles) {
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
      if ((lane & 7) == 0 && (lane >> 3) < tiles)
        sh.seg[(t0 + (lane >> 3)) * SV_WAVES + wave] = ldexp(s, down_by);  // (segments past the row's end: zero)
    };
    store(0, TILES);
    if constexpr (MORE) {
      for (int t0 = TILES; t0 * SV_WAVES < n_blocks; t0 += 8) {  // (t0 < 64: n_blocks <= SV_MAX_SEGS)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          s8[i] = 0.0;
          if ((t0 + i) * SV_WAVES + wave < n_blocks) {
            double m[4];
            more(t0 + i, true, m);
            s8[i] = (m[0] + m[1]) + (m[2] + m[3]);
          }
          asm volatile("" : "+v"(s8[i]));
        }
        store(t0, min(8, SV_MAX_SEGS / SV_WAVES - t0));
      }
    }
    __syncthreads();
    tok = -1;
    Hit h;
    if (!find_segment(sh.seg, n_blocks, MORE ? (n_blocks + 63) >> 6 : (TILES * SV_WAVES + 63) / 64, u, 2.0 * SV_BLOCK * MASS_FLOOR, lane, h)) return false;
    if (wave == h.seg % SV_WAVES) {            // (the segment's own wave: it holds the masses, of which one is above the floor)
      const double target = ldexp(h.target, -down_by);
      int tail = -1;
      double m[4] = {ex[0][0], ex[0][1], ex[0][2], ex[0][3]};
#pragma unroll
      for (int t = 1; t < TILES; ++t)
        if (h.seg / SV_WAVES == t) {           // (wave-uniform)
#pragma unroll
          for (int i = 0; i < 4; ++i) m[i] = ex[t][i];
        }
      if constexpr (MORE) {
        if (h.seg / SV_WAVES >= TILES) more(h.seg / SV_WAVES, false, m);
      }
      find_token(m, h.seg * SV_BLOCK + 4 * lane, 0.0, target, MASS_FLOOR, tok, tail);
      if (tok < 0) tok = tail;                 // rounding left the target at the segment's end: its last token with mass
    }
    return true;
  }
};

// Largest score of a row, then Z = sum_v exp((l_v - max) / T), both uniform over the workgroup, for rows of any kind
__device__ __forceinline__ void row_max_and_z(const float* __restrict__ L, int V, Temp& temp, DrawShared& sh, int tid, double& Z) {
  const int lane = tid & 63, wave = wave_of(tid);
  float mx = -INFINITY;
  wave_blocks<0>(V, wave, [&](int blk, int) {
    const f32x4 l = load_row4(L, blk, lane, V, -INFINITY);
    mx = fmaxf(mx, fmaxf(fmaxf(l[0], l[1]), fmaxf(l[2], l[3])));
  });
  mx = wave_max(mx);
  if (lane == 0) sh.redf[wave] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < SV_WAVES; ++w) mx = fmaxf(mx, sh.redf[w]);
  temp.below(mx);
  double zp = 0.0;
  wave_blocks<0>(V, wave, [&](int blk, int) {
    const int v = blk * SV_BLOCK + 4 * lane;
    double m[4];
    temp.mass4<true>(load_row4(L, blk, lane, V, -INFINITY), m);
#pragma unroll
    for (int e = 0; e < 4; ++e) zp += v + e < V ? m[e] : 0.0;
  });
  zp = wave_sum_d(zp);
  __syncthreads();  // (the sums of the registers' attempt have been read)
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
template <int TILES, bool MORE, bool SHIFT>
__global__ void __launch_bounds__(SV_THREADS) verify_sample_kernel(
    const float* __restrict__ logits, const int32_t* __restrict__ voted, const float* __restrict__ draft_probs,
    const int32_t* __restrict__ spec_len, const int32_t* __restrict__ greedy, int B, int k_max, int M, int V,
    double temperature, double inv_temperature, double k, double k_lo, uint32_t seed_lo, uint32_t seed_hi, uint32_t step_lo, uint32_t step_hi,
    int32_t* __restrict__ sampled, int32_t* dev_status) {
  __shared__ DrawShared sh;
  __shared__ int s_int[2];  // rows before this sequence, bad flag
  const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = wave_of(tid);
  int32_t* out = sampled + (size_t)b * (k_max + 1) + j;

  PowerLoad power;
  power.ask(tid);
  const int k_b = spec_len[b], first = greedy[(size_t)b * (k_max + 1)];
  const int x = j < k_max ? voted[(size_t)b * k_max + j] : -1;  // (looked at below k_b only)
  int row = j, bad = 0;  // rows of the sequences before b
  if (b <= 256) {        // every wave for itself, nobody waits
    int n[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) n[i] = i * 64 < b ? spec_len[min(i * 64 + lane, b)] : 0;
    int part = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i * 64 + lane < b) {
        bad |= n[i] < 0 || n[i] > k_max;
        part += n[i] + 1;
      }
    row += wave_sum_i(part);
    bad = __any(bad);
  } else {
    if (tid < 2) s_int[tid] = 0;
    __syncthreads();
    int part = 0;
    for (int i = tid; i < b; i += SV_THREADS) {
      const int n = spec_len[i];
      if (n < 0 || n > k_max) bad = 1;
      part += n + 1;
    }
    if (part) atomicAdd(&s_int[0], part);  // (integer sum: order-free)
    if (bad) atomicOr(&s_int[1], 1);
    __syncthreads();
    row += s_int[0];
    bad = s_int[1];
  }
  row = __builtin_amdgcn_readfirstlane(row);
  const bool seq_ok = !bad && k_b >= 0 && k_b <= k_max && first >= 0;
  if (!seq_ok || j > k_b || row >= M) {  // (whole workgroup)
    if (tid == 0) {
      *out = -1;
      if (seq_ok && j <= k_b && dev_status) atomicOr(dev_status, MN_DEV_SPEC_LEN);  // rows do not add up to M
    }
    return;
  }
  const float* L = logits + (size_t)row * V;
  const float* Q = j < k_b ? draft_probs + ((size_t)b * k_max + j) * V : nullptr;
  const bool in_vocab = Q && x >= 0 && x < V;
  float l_x = 0.f, q_x = 0.f;
  if (in_vocab) {
    l_x = L[x];
    q_x = Q[x];
  }
  Temp temp(temperature, inv_temperature, k, k_lo, sh);
  double u_acc = 0.0, u_res = 0.0;
  auto uniforms = [&]() { position_uniforms((uint32_t)b, (uint32_t)j, step_lo, step_hi, 0u, seed_lo, seed_hi, u_acc, u_res); };
  // does the speculated token survive?  (mass_x of Z)
  auto survives = [&](double mass_x, double Z) {
    const double ox = mass_x / Z, qx = (double)q_x;
    return qx <= ox || u_acc < ox / qx;
  };

  // ---- where it does not, a token from max(0, o - q); without q (position k_b) from o.  When nothing of o lies above q (a q that
  // sums above 1) the replacement comes from o without the rejected token, so that it still differs from what
  // it replaces (the acceptance reads "first entry that differs" as the first rejection); and when all of o
  // sits on that token there is nothing else to emit: it stays ----
  if constexpr (TILES > 0) {
    RowRegs<TILES, MORE, SHIFT> regs;
    if (regs.load(L, Q, V, temp, power, sh, tid)) {
      uniforms();
      if (in_vocab) {
        Temp whole = temp;
        whole.relative_to(regs.e_all, (double)regs.e_all * 256.0 / temp.k);
        if (survives(whole.mass<false>(SHIFT ? l_x - regs.shift : l_x), regs.Z)) {  // (whole workgroup: all of it is uniform)
          if (tid == 0) *out = x;
          return;
        }
      }
      if (Q) {  // masses of o - q, times Z and relative to the wave's power of two
        constexpr int HALF = TILES <= 4 ? TILES : (TILES + 1) / 2;
#pragma unroll
        for (int h = 0; h < TILES; h += HALF) {
          f32x4 q[HALF];
#pragma unroll
          for (int t = 0; t < HALF; ++t) q[t] = regs.ask(Q, min(h + t, TILES - 1), wave, lane, V);
#pragma unroll
          for (int t = 0; t < HALF && h + t < TILES; ++t) {
            if (regs.may_end(h + t) && V & 3) q[t] = regs.in_place(q[t], h + t, wave, lane, V);
            asm volatile("" : "+v"(q[t]));
#pragma unroll
            for (int e = 0; e < 4; ++e) regs.ex[h + t][e] = fmax(0.0, fma(-(double)q[t][e], regs.z_wave, regs.ex[h + t][e]));
            in_turn(regs.ex[h + t][0], regs.ex[h + t][1], regs.ex[h + t][2], regs.ex[h + t][3]);
            regs.clear_past_end(h + t, wave, lane, V);
          }
        }
      }
      int tok;
      auto more = [&](int t, bool, double (&m)[4]) {
        f32x4 q = {0.f, 0.f, 0.f, 0.f};
        if (Q) q = regs.ask(Q, t, wave, lane, V);
        regs.far(L, t, wave, lane, V, temp, m);
        if (Q) {
          q = regs.in_place(q, t, wave, lane, V);
          const bool last = ((t * SV_WAVES + wave) + 1) * SV_BLOCK > V;  // (wave-uniform)
#pragma unroll
          for (int e = 0; e < 4; ++e) m[e] = last && (t * SV_WAVES + wave) * SV_BLOCK + 4 * lane + e >= V ? 0.0 : fmax(0.0, fma(-(double)q[e], regs.z_wave, m[e]));
        }
      };
      if (regs.draw(V, u_res, regs.down, sh, tid, tok, more)) {
        if (tok >= 0 && lane == 0) *out = tok;  // (one wave)
        return;
      }
    }
    __syncthreads();                            // (the general form starts over)
  } else {
    power.store(sh, tid);
    __syncthreads();
  }
  double Z;
  row_max_and_z(L, V, temp, sh, tid, Z);
  uniforms();
  if (in_vocab && survives(temp.mass<true>(l_x), Z)) {
    if (tid == 0) *out = x;
    return;
  }
  const double inv_z = 1.0 / Z;  // (Z >= 1: the largest score contributes exp(0))
  auto o4 = [&](int blk, double (&o)[4]) {  // probabilities of a block's tokens, recomputed from the scores
    const int v = blk * SV_BLOCK + 4 * lane;
    const f32x4 l = load_row4(L, blk, lane, V, -INFINITY);
    temp.mass4<true>(l, o);
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = v + e < V ? div_by(o[e], Z, inv_z) : 0.0;
  };
  int tok = cdf_draw([&](int blk, double (&m)[4]) {
                     o4(blk, m);
                     if (Q) {
                       const f32x4 q = load_row4(Q, blk, lane, V, 0.f);
#pragma unroll
                       for (int e = 0; e < 4; ++e) m[e] = fmax(0.0, m[e] - (double)q[e]);
                     }
                   },
                   V, u_res, sh, tid);
  if (Q && tok < 0) {
    tok = cdf_draw([&](int blk, double (&m)[4]) {
                     o4(blk, m);
#pragma unroll
                     for (int e = 0; e < 4; ++e)
                       if (blk * SV_BLOCK + 4 * lane + e == x) m[e] = 0.0;
                   },
                   V, u_res, sh, tid);
    if (tok < 0) tok = x;
  }
  if (tid == 0) *out = tok;
}

// One workgroup per sequence: token ~ q = softmax(scores / T) of a drafting SSM, and q itself in fp32.
// The draw is taken from the fp32 values that are written out, so what the verifier is later told is
// exactly the distribution the token came from.
template <int TILES, bool MORE, bool SHIFT>
__global__ void __launch_bounds__(SV_THREADS) draft_sample_kernel(const float* __restrict__ logits, int V,
                                                                  double temperature, double inv_temperature, double k, double k_lo,
                                                                  uint32_t seed_lo, uint32_t seed_hi,
                                                                  uint32_t step_lo, uint32_t step_hi, uint32_t consumer,
                                                                  uint32_t t_pos, int32_t* __restrict__ tokens,
                                                                  long token_stride, float* __restrict__ probs,
                                                                  long probs_stride) {
  __shared__ DrawShared sh;
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = wave_of(tid);
  const float* L = logits + (size_t)b * V;
  int32_t* out = tokens + (size_t)b * token_stride;
  float* P = probs ? probs + (size_t)b * probs_stride : nullptr;
  PowerLoad power;
  power.ask(tid);
  Temp temp(temperature, inv_temperature, k, k_lo, sh);
  auto uniform = [&]() {
    double u_unused, u;
    position_uniforms((uint32_t)b, t_pos, step_lo, step_hi, consumer, seed_lo, seed_hi, u_unused, u);
    return u;
  };
  auto write = [&](int blk, const double (&m)[4]) {
    if (!P) return;
    const int v = blk * SV_BLOCK + 4 * lane;
    if ((blk + 1) * SV_BLOCK <= V || v + 3 < V) {
      *reinterpret_cast<f32x4_u*>(P + (size_t)blk * SV_BLOCK + 4 * lane) = (f32x4_u){(float)m[0], (float)m[1], (float)m[2], (float)m[3]};
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (v + e < V) P[v + e] = (float)m[e];
    }
  };
  if constexpr (TILES > 0) {
    RowRegs<TILES, MORE, SHIFT> regs;
    if (regs.load(L, nullptr, V, temp, power, sh, tid)) {
      const double inv_z = regs.dead ? 0.0 : 1.0 / regs.z_wave;
#pragma unroll
      for (int t = 0; t < TILES; ++t) {
#pragma unroll
        for (int e = 0; e < 4; ++e) regs.ex[t][e] = (double)(float)div_by(regs.ex[t][e], regs.z_wave, inv_z);
        in_turn(regs.ex[t][0], regs.ex[t][1], regs.ex[t][2], regs.ex[t][3]);
        write(t * SV_WAVES + wave, regs.ex[t]);
      }
      int tok;
      auto more = [&](int t, bool first, double (&m)[4]) {
        regs.far(L, t, wave, lane, V, temp, m);
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] = (double)(float)div_by(m[e], regs.z_wave, inv_z);
        if (first) write(t * SV_WAVES + wave, m);
      };
      if (!regs.draw(V, uniform(), 0, sh, tid, tok, more)) {
        if (tid == 0) *out = -1;
      } else if (tok >= 0 && lane == 0) {  // (one wave)
        *out = tok;
      }
      return;
    }
    __syncthreads();                       // (the general form starts over)
  } else {
    power.store(sh, tid);
    __syncthreads();
  }
  double Z;
  row_max_and_z(L, V, temp, sh, tid, Z);
  const double inv_z = 1.0 / Z;
  auto q4 = [&](int blk, double (&m)[4]) {  // the fp32 probabilities of a block's tokens
    const int v = blk * SV_BLOCK + 4 * lane;
    const f32x4 l = load_row4(L, blk, lane, V, -INFINITY);
    temp.mass4<true>(l, m);
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = v + e < V ? (double)(float)div_by(m[e], Z, inv_z) : 0.0;
  };
  if (P)
    wave_blocks<0>(V, wave, [&](int blk, int) {
      double m[4];
      q4(blk, m);
      write(blk, m);
    });
  const int tok = cdf_draw([&](int blk, double (&m)[4]) {
                     const int v = blk * SV_BLOCK + 4 * lane;
                     if (P && v + 3 < V) {  // (this thread wrote them itself: cheaper than the exponentials again)
                       const f32x4_u q = *reinterpret_cast<const f32x4_u*>(P + v);
                       m[0] = (double)q[0]; m[1] = (double)q[1]; m[2] = (double)q[2]; m[3] = (double)q[3];
                     } else {
                       q4(blk, m);
                     }
                   },
                   V, uniform(), sh, tid);
  if (tid == 0) *out = tok;
}

// 1 / T where both are comfortably normal numbers, 0 otherwise (the kernels then divide)
static double temperature_reciprocal(double T) { return T > 0x1p-100 && T < 0x1p100 ? 1.0 / T : 0.0; }
// 256 / (T ln2) in two pieces (about 104 bits: scores far from zero beside T multiply its error)
struct StepsPerScore {
  double k, k_lo;
  explicit StepsPerScore(double T) {
    const double c = 0x1.71547652b82fep+8, c_lo = 0x1.777d0ffda0d24p-48;  // 256 / ln2
    k = c / T;
    k_lo = (std::fma(-k, T, c) + c_lo) / T;
  }
};

// Tiles of 4096 tokens that a row's exponentials take in registers: an instance for every number of them, since each computes all of its tiles (a branch around
// those that a wave does not have costs 0.7 us at 32000 tokens; with instances of 1, 2, 4 and 8 tiles alone 16 drafted tokens of 8193, 17000 and 25000 took 9.1, 12.4 and
// 12.2 us, now 7.6, 9.2 and 10.9).  0: the general form.  Beyond 32768 tokens the first tiles are in registers, up to the segments that the shared array
// holds.
constexpr int SV_MAX_FAR = SV_MAX_SEGS * SV_BLOCK;
static int reg_tiles(int V, double T, double inv) {
  // (at 2^90 and more, 690 T below a largest score near the type's lowest value is no float: a cut score would stand level with it)
  if (V < 4 || V > SV_MAX_FAR || inv == 0.0 || T >= 0x1p90) return 0;
  return min((V + SV_TILE - 1) / SV_TILE, SV_REG_TILES + 1);
}
// FAR: tiles in registers beyond 32768 tokens.  144 positions of 50272 tokens 26.2 us with six, 28.6 with four, 25.0 with eight, which keep five registers in scratch memory
// (an earlier build of them, with more there, took 35.6), 48.4 in the general form; 16 drafted tokens 20.6 with eight, 22.3 with six, 24.4 with four, 41.5 in the general form.
// Temperatures below SV_LOW_T, whose scores may be 2^38 steps of the exponentials' table from zero (a score of 709 there, of 20 at T 2.7e-8), take them less the
// row's largest, which the waves wait for: 32000 tokens at T 1e-9, 144 positions 13.4 us and 16 drafted tokens 11.9 (37.1 and 33.4 in the general form after an attempt
// that found it out, 12.9 and 11.7 without the row's largest at 1e-6), 50272 tokens 28.4 and 22.1 (56.6 and 49.6; 26.4 and 21.3).  Rows of 3, 5, 6 and 7 tiles go with the next instance.
constexpr double SV_LOW_T = 0x1p-20;
#define MN_ROW_KERNEL(K, FAR, V, T, INV)                                                                                               \
  [&] {                                                                                                                                \
    const int tiles = reg_tiles(V, T, INV);                                                                                            \
    if (tiles > 0 && T < SV_LOW_T)                                                                                                     \
      return tiles <= 2 ? K<2, false, true> : tiles <= 4 ? K<4, false, true> : tiles <= 8 ? K<8, false, true> : K<FAR, true, true>;    \
    switch (tiles) {                                                                                                                   \
      case 0: return K<0, false, false>;                                                                                               \
      case 1: return K<1, false, false>;                                                                                               \
      case 2: return K<2, false, false>;                                                                                               \
      case 3: return K<3, false, false>;                                                                                               \
      case 4: return K<4, false, false>;                                                                                               \
      case 5: return K<5, false, false>;                                                                                               \
      case 6: return K<6, false, false>;                                                                                               \
      case 7: return K<7, false, false>;                                                                                               \
      case 8: return K<8, false, false>;                                                                                               \
      default: return K<FAR, true, false>;                                                                                             \
    }                                                                                                                                  \
  }()
static_assert(SV_REG_TILES == 8, "an instance for every number of tiles");

void launch_verify_sample(const float* logits, const int32_t* voted, const float* draft_probs, const int32_t* spec_len,
                          const int32_t* greedy, int B, int k_max, int M, int V, double temperature, uint64_t seed,
                          uint64_t step, int32_t* sampled, int32_t* dev_status, hipStream_t st) {
  if (B <= 0) return;
  const double inv = temperature_reciprocal(temperature);
  const StepsPerScore steps(temperature);
  auto* kernel = MN_ROW_KERNEL(verify_sample_kernel, 6, V, temperature, inv);
  kernel<<<dim3(k_max + 1, B), SV_THREADS, 0, st>>>(
      logits, voted, draft_probs, spec_len, greedy, B, k_max, M, V, temperature, inv, steps.k, steps.k_lo,
      (uint32_t)seed, (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32), sampled, dev_status);
}

void launch_draft_sample(const float* logits, int B, int V, double temperature, uint64_t seed, uint64_t step, int ssm,
                         int t_pos, int32_t* tokens, long token_stride, float* probs, long probs_stride, hipStream_t st) {
  if (B <= 0) return;
  const double inv = temperature_reciprocal(temperature);
  const StepsPerScore steps(temperature);
  auto* kernel = MN_ROW_KERNEL(draft_sample_kernel, 8, V, temperature, inv);
  kernel<<<B, SV_THREADS, 0, st>>>(logits, V, temperature, inv, steps.k, steps.k_lo, (uint32_t)seed,
                                   (uint32_t)(seed >> 32), (uint32_t)step, (uint32_t)(step >> 32), (uint32_t)(1 + ssm),
                                   (uint32_t)t_pos, tokens, token_stride, probs, probs_stride);
}

int verify_sample_max_vocab() { return SV_MAX_VOCAB; }

}  // namespace mn
