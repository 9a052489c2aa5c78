// Device helpers of the GSQ kernels: Philox4x32-10, the noise transforms, bf16 rounding.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gsq {

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds, each multiplying words
// 0 and 2 by the round multipliers and mixing the 64-bit products' halves with the other
// words and the round key; the key advances by the two Weyl constants between rounds.
struct U4 { uint32_t x, y, z, w; };

// x ^ y ^ z in one instruction, which the compiler does not form by itself (truth table 0x96).  With
// the key's word it takes 20 of a Philox call's 60-odd instructions away.
__device__ __forceinline__ uint32_t xor3(uint32_t x, uint32_t y, uint32_t z) {
  return __builtin_amdgcn_bitop3_b32(x, y, z, 0x96);
}

__device__ __forceinline__ U4 philox10(U4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
    c = U4{xor3((uint32_t)(p1 >> 32), c.y, k0), (uint32_t)p1, xor3((uint32_t)(p0 >> 32), c.w, k1),
           (uint32_t)p0};
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c;
}

// Noise layout: the four coordinates e0 .. e0+3 of an aligned chunk (e0 = e - e mod 4) read
// their 4K values, coordinate e0+q / level k at flat position f = q K + k, from K Philox calls:
// call j has counter (e0 mod 2^32, e0 >> 32, t, tag*256 + j) and position f takes word
// f mod 4 of call f div 4.  tag = sample*256 + stream, stream 0 = step noise, 1 = initial logit
// noise, sample = index of an independent draw within one step; key = seed.
__device__ __forceinline__ U4 noise_words(uint64_t seed, uint64_t e0, uint32_t t, uint32_t tag,
                                          uint32_t j) {
  return philox10(U4{(uint32_t)e0, (uint32_t)(e0 >> 32), t, tag * 256u + j}, (uint32_t)seed,
                  (uint32_t)(seed >> 32));
}

__device__ __forceinline__ uint32_t word_of(const U4& w, int r) {
  return r == 0 ? w.x : r == 1 ? w.y : r == 2 ? w.z : w.w;
}

// u = (top 23 bits + 1/2) * 2^-23, exact in fp32, in [2^-24, 1 - 2^-24]: the float with
// mantissa m = x >> 9 and exponent 0 is 1 + m 2^-23; subtracting 1 - 2^-24 (exact, the result
// has at most 24 significant bits) leaves (m + 1/2) 2^-23.
__device__ __forceinline__ float uniform01(uint32_t x) {
  return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, x, 9)) - 0x1.fffffep-1f;
}

// fp64 functions for the arguments met here, to about 1 ulp of fp64: the library's, which also serve
// every other argument, take 98, 42 and 22 vector instructions, these 26, 20 and 12.  The reductions
// are those of Cody and Waite, "Software Manual for the Elementary Functions" (1980): ln through
// (m - 1) / (m + 1), exp through a multiple of ln 2 in two words; the root is Goldschmidt's coupled
// iteration (1964).  Polynomials by interpolation at Chebyshev points, with coefficients of our own.

// ln x of a positive normal x: x = 2^e m with m in [sqrt(1/2), sqrt(2)), f = m - 1,
// s = f / (2 + f), ln m = f - s (f - z P(z)) with z = s^2 and 2 atanh(s) = 2 s + s z P(z); the
// polynomial is within 5e-18 of it on z <= 0.02945.
__device__ __forceinline__ double log_pos(double x) {
  double m = __builtin_amdgcn_frexp_mant(x);
  const int low = m < 0x1.6a09e667f3bcdp-1 ? 1 : 0;
  const int e = __builtin_amdgcn_frexp_exp(x) - low;
  m = __builtin_ldexp(m, low);
  const double f = m - 1.0, d = m + 1.0;
  double r = __builtin_amdgcn_rcp(d);
  r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
  r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
  const double s = f * r, z = s * s;
  double p = 0x1.2b5b5fb2eac92p-3;
  p = __builtin_fma(p, z, 0x1.39fe208c33457p-3);
  p = __builtin_fma(p, z, 0x1.7462b69705382p-3);
  p = __builtin_fma(p, z, 0x1.c71c62debf86bp-3);
  p = __builtin_fma(p, z, 0x1.2492492df6947p-2);
  p = __builtin_fma(p, z, 0x1.99999999952b2p-2);
  p = __builtin_fma(p, z, 0x1.5555555555558p-1);
  return __builtin_fma((double)e, 0x1.62e42fefa39efp-1,
                       __builtin_fma(-s, __builtin_fma(-z, p, f), f));
}

// e^x of x <= 0 (NaN stays NaN): x = t ln 2 + r with |r| <= ln(2) / 2, e^r = 1 + r + r^2 Q(r), the
// polynomial within 1.3e-17; below -1100 the result is 0 as at -1100.
__device__ __forceinline__ double exp_nonpos(double x) {
  x = x < -1100.0 ? -1100.0 : x;
  const double t = __builtin_rint(x * 0x1.71547652b82fep+0);
  double r = __builtin_fma(-t, 0x1.62e42fee00000p-1, x);
  r = __builtin_fma(-t, 0x1.a39ef35793c76p-33, r);
  double q = 0x1.af38a9b0ec855p-26;
  q = __builtin_fma(q, r, 0x1.289185613a3d6p-22);
  q = __builtin_fma(q, r, 0x1.71de0dae63bb3p-19);
  q = __builtin_fma(q, r, 0x1.a019b90d2ae7ap-16);
  q = __builtin_fma(q, r, 0x1.a01a01a7c41d5p-13);
  q = __builtin_fma(q, r, 0x1.6c16c1788bd90p-10);
  q = __builtin_fma(q, r, 0x1.11111111109b3p-7);
  q = __builtin_fma(q, r, 0x1.5555555553d63p-5);
  q = __builtin_fma(q, r, 0x1.5555555555556p-3);
  q = __builtin_fma(q, r, 0x1.0000000000001p-1);
  const double y = 1.0 + __builtin_fma(q * r, r, r);
  return __builtin_ldexp(y, (int)t);
}

// Square root (0 and infinity as they are, NaN for what is below 0); below the normal range to fp32's
// accuracy at least.  One coupled step of Newton for the root and its reciprocal, one for the root.
__device__ __forceinline__ double sqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double c = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, c, g);
  h = __builtin_fma(h, c, h);
  g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
  return x == 0.0 || x == __builtin_inf() ? x : g;
}

// Gumbel(0,1) sample -ln(-ln u): evaluated in fp64 and rounded once to fp32.
__device__ __forceinline__ float gumbel_exact(uint32_t x) {
  const double u = (double)uniform01(x);
  return (float)(-log_pos(-log_pos(u)));
}

// Gumbel(0,1) sample with the hardware base-2 logarithm:
// -ln(-ln u) = -ln2 * log2(-ln2 * log2 u).
__device__ __forceinline__ float gumbel_fast(uint32_t x) {
  constexpr float kLn2 = 0.69314718055994531f;
  const float u = uniform01(x);
  const float nl = __builtin_amdgcn_logf(u) * -kLn2;   // -ln u > 0
  return __builtin_amdgcn_logf(nl) * -kLn2;
}

// Logistic(0,1) sample ln u - ln(1 - u), the noise of a two-value relaxation with logits
// {-l, l}: its softmax sees the two Gumbel values only through their difference, which has this
// law.  1 - u is exact in fp32 (u has at most 24 significant bits below 1).  Exact: evaluated in
// fp64 and rounded once to fp32; fast: ln2 (log2 u - log2(1 - u)) with the hardware logarithm.
__device__ __forceinline__ float logistic_exact(uint32_t x) {
  const float u = uniform01(x);
  return (float)(log_pos((double)u) - log_pos((double)(1.0f - u)));
}

__device__ __forceinline__ float logistic_fast(uint32_t x) {
  constexpr float kLn2 = 0.69314718055994531f;
  const float u = uniform01(x);
  return (__builtin_amdgcn_logf(u) - __builtin_amdgcn_logf(1.0f - u)) * kLn2;
}

// Transform of a noise word: Gumbel values for categoricals, logistic values for binary pairs.
enum NoiseKind { kGumbel = 0, kLogistic = 1 };

template <int kKind, bool kExact>
__device__ __forceinline__ float noise_value(uint32_t x) {
  if constexpr (kKind == kLogistic) {
    if constexpr (kExact) return logistic_exact(x); else return logistic_fast(x);
  } else {
    if constexpr (kExact) return gumbel_exact(x); else return gumbel_fast(x);
  }
}

// The 4 x K noise values of the chunk starting at e0 (a multiple of 4) at step t.
template <int K, bool kExact, int kKind = kGumbel>
__device__ __forceinline__ void draw_chunk(float (&g)[4][K], uint64_t seed, uint64_t e0, uint32_t t,
                                           uint32_t sample) {
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const U4 w = noise_words(seed, e0, t, sample * 256u, (uint32_t)j);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      g[(4 * j + r) / K][(4 * j + r) % K] = noise_value<kKind, kExact>(word_of(w, r));
  }
}

// The K noise values of one coordinate e at step t (any e; draws only the calls it needs).
template <int K, bool kExact, int kKind = kGumbel>
__device__ __forceinline__ void draw_one(float (&g)[K], uint64_t seed, uint64_t e, uint32_t t) {
  const uint64_t e0 = e & ~(uint64_t)3;
  const int q = (int)(e & 3);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int f = q * K + k;
    g[k] = noise_value<kKind, kExact>(word_of(noise_words(seed, e0, t, 0u, (uint32_t)(f >> 2)), f & 3));
  }
}

// float -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint16_t bf16_rne(float f) {
  uint32_t b = __float_as_uint(f);
  b += 0x7FFFu + ((b >> 16) & 1u);
  return (uint16_t)(b >> 16);
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// x shifted up by n lanes within each 16-lane row (lanes below the row start read 0).
template <int kCtrl>
__device__ __forceinline__ double dpp_shr(double x) {
  const uint64_t b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, kCtrl, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), kCtrl, 0xF, 0xF, false);
  return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// x from lane 15 of the previous 16-lane row (kCtrl = row broadcast 15) or from lane 31
// (row broadcast 31), added only in the rows of kRows; other lanes read 0.
template <int kCtrl, int kRows>
__device__ __forceinline__ double dpp_bcast(double x) {
  const uint64_t b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, kCtrl, kRows, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), kCtrl, kRows, 0xF, false);
  return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

// Sum over the wavefront in a fixed order, left in lane 63: prefix sums within each 16-lane
// row (shifts by 1, 2, 4, 8), then row 0's total into row 1 and row 2's into row 3, then the
// first half's total into the second half.
__device__ __forceinline__ double wave_sum_to_lane63(double x) {
  x += dpp_shr<0x111>(x);
  x += dpp_shr<0x112>(x);
  x += dpp_shr<0x114>(x);
  x += dpp_shr<0x118>(x);
  x += dpp_bcast<0x142, 0xA>(x);
  x += dpp_bcast<0x143, 0xC>(x);
  return x;
}

}  // namespace gsq
